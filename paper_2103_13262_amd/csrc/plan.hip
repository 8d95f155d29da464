// Counting, offsets and the stable position of every assignment inside its expert's segment
// (Section 3.2: the samples per expert are counted first and the buffer offsets follow from
// the counts; Section 4: the samples of one expert lie contiguously).  Integer work only.
//
//   plan_hist  : per chunk of assignments, an LDS histogram over experts (batches of more than kOwnCounts assignments only).
//   plan_place : workgroup 0 writes the tables - counts, offsets, tile prefix tables for four row-tile heights, size
//                classes; workgroup 1 the experts in order of descending count and the control block; every other workgroup
//                places the assignments of one chunk.  All of them work out the counts and offsets they need for themselves (from the
//                chunk histograms, or from the indices where those are few), so that the placing does not wait for a
//                launch of one workgroup in front of it.  Ranks inside a wavefront come from ballots (lanes that hold the same
//                expert are found bit by bit), so rows keep assignment order.
// Bound by latency.  With the tables in a launch of one workgroup and the placing behind it: 12.4 us at 8192 assignments and 16
// experts, 17.2 us at 200 and 256, 21.5 us at 16384 and 256, 29.0 us at 65536 and 32; then
// 8.8, 8.4, 14.2 and 11.0 us; with the order in a workgroup of its own beside the tables 0.6 us less for few experts, 1.8 less for 256 (gate and plan of 200 tokens
// 17.4 -> 15.5) and 3.4 less for 600.
#include "common.h"

namespace moe {

constexpr int kThreads = 1024, kWaves = kThreads / 64;
// Assignments up to which every workgroup counts them itself; more are counted by plan_hist first.  Own counts against chunk
// histograms, us: 4 experts (whose few counters the atomics meet on) 8.8 / 10.6 at 4096 assignments, 12.0 / 10.6 at 8192; 16 experts 10.1 / 10.6
// at 8192, 11.7 / 10.8 at 12288; 256 experts 12.6 / 15.0 at 8192, 15.3 / 14.9 at 16384; 1024 experts 20.2 / 22.4 at 8192, 27.4 / 24.8 at 32768.
constexpr int kOwnCounts = 8 * 1024;

__global__ __launch_bounds__(kThreads) void plan_hist(const int32_t* __restrict__ idx, long M, int E, int chunk, int32_t* __restrict__ hist)
{
    __shared__ int sh[kMaxE];
    for (int e = threadIdx.x; e < E; e += kThreads) sh[e] = 0;
    __syncthreads();
    const long base = (long)blockIdx.x * chunk, end = min(base + chunk, M);
    for (long a = base + threadIdx.x; a < end; a += kThreads) {
        const int e = idx[a];
        if (e >= 0 && e < E) atomicAdd(&sh[e], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kThreads) hist[(size_t)blockIdx.x * E + e] = sh[e];
}

// Exclusive scans of NV ints per thread over a 1024-thread workgroup, all at once (v[i] -> sum of v[i] over the
// threads below); `total[i]` receives the sums.  Threads n_used and above hold zeros: their wavefronts skip the
// shuffles (the LDS crossbar that carries them is shared by all sixteen).
template <int NV>
__device__ __forceinline__ void block_excl_scan_1024(int (&v)[NV], int (*s_wave)[NV] /*[16][NV]*/, int (&total)[NV], int n_used)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) inc[i] = v[i];
    if (wave * 64 < n_used) {
        for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int o = __shfl_up(inc[i], off, 64);
                if (lane >= off) inc[i] += o;
            }
        }
    }
    if (lane == 63) {
#pragma unroll
        for (int i = 0; i < NV; ++i) s_wave[wave][i] = inc[i];
    }
    __syncthreads();
    int wbase[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) wbase[i] = total[i] = 0;
    for (int w = 0; w * 64 < n_used; ++w) {           // (a wavefront's NV sums are read together)
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = s_wave[w][i];
            if (w < wave) wbase[i] += c;
            total[i] += c;
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = wbase[i] + inc[i] - v[i];
}

// hist == nullptr: every workgroup counts the assignments itself.
__global__ __launch_bounds__(kThreads) void plan_place(const int32_t* __restrict__ idx, const int32_t* __restrict__ hist, int nb, int chunk,
                                                       int E, int nbits, long M, int32_t* __restrict__ counts,
                                                       int32_t* __restrict__ offsets, int32_t* __restrict__ tileP,
                                                       int32_t* __restrict__ order, int32_t* __restrict__ cls,
                                                       int32_t* __restrict__ control, int32_t* __restrict__ arrive, int arrive_words, int32_t* __restrict__ pos,
                                                       int32_t* __restrict__ perm)
{
    extern __shared__ __align__(16) int smem_plan[];
    const int Ep = (E + 3) & ~3;
    int* const s_total = smem_plan;                 // [Ep] rows of every expert
    int* const s_below = s_total + Ep;              // [Ep] those in the chunks before this workgroup's; then the next free row
    int* const s_w = s_below + Ep;                  // [kWaves][Ep] (placing)
    __shared__ int s_wave[kWaves * (3 + kNumTileHeights)];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool tables = blockIdx.x < 2;             // workgroup 0: counts, offsets, tiles, size classes; 1: the experts in order
    const int b = (int)blockIdx.x - 2;              // this workgroup's chunk
    const long base = (long)b * chunk;
    auto index = [&](long a) {                      // (an index out of range cannot come from the gate kernels)
        int e = -1;
        if (a < M) { e = idx[a]; if (e < 0 || e >= E) e = -1; }
        return e;
    };
    int ev = tables ? -1 : index(base + tid);       // first round, on its way while the counts are taken
    // the control words of the grouped products
    if (blockIdx.x == 1 && tid < kCtlWords) control[tid] = 0;
    if (blockIdx.x == gridDim.x - 1)                // the counters of the backward pass's sums
        for (int i = tid; i < arrive_words; i += kThreads) arrive[i] = 0;
    for (int e = tid; e < 2 * Ep; e += kThreads) s_total[e] = 0;
    __syncthreads();
    if (hist) {
        int width = 1;
        while (width < E) width <<= 1;
        const int e = tid & (width - 1), groups = kThreads / width;
        if (e < E) {
            int total = 0, below = 0;
            for (int r0 = tid / width; r0 < nb; r0 += 8 * groups) {     // eight rows in flight
                int v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = hist[(size_t)min(r0 + u * groups, nb - 1) * E + e];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int r = r0 + u * groups;
                    if (r < nb) { total += v[u]; if (r < b) below += v[u]; }
                }
            }
            atomicAdd(&s_total[e], total);
            if (below) atomicAdd(&s_below[e], below);
        }
    } else {
        for (long a0 = 0; a0 < M; a0 += 8 * kThreads) {
            int v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = index(a0 + u * kThreads + tid);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (v[u] >= 0) {
                    atomicAdd(&s_total[v[u]], 1);
                    if (a0 + u * kThreads + tid < base) atomicAdd(&s_below[v[u]], 1);
                }
        }
    }
    __syncthreads();

    if (!tables) {
        int sc[1] = {tid < E ? s_total[tid] : 0}, total[1];
        block_excl_scan_1024<1>(sc, (int (*)[1])s_wave, total, E);
        if (tid < E) s_below[tid] += sc[0];
        for (long a0 = base; a0 < min(base + chunk, M); a0 += kThreads) {
            const long a = a0 + tid;
            const int next = a0 + kThreads < base + chunk ? index(a + kThreads) : -1;
            for (int i = tid; i < kWaves * Ep; i += kThreads) s_w[i] = 0;
            __syncthreads();
            const bool valid = ev >= 0;
            unsigned long long mask = __ballot(valid);
            for (int bit = 0; bit < nbits; ++bit) {
                const bool on = valid && ((ev >> bit) & 1);
                const unsigned long long bal = __ballot(on);
                mask &= on ? bal : ~bal;
            }
            const int rank = __popcll(mask & ((1ull << lane) - 1ull));
            if (valid && rank == 0) s_w[wave * Ep + ev] = __popcll(mask);
            __syncthreads();
            if (tid < E) {
                int run = s_below[tid], c[kWaves];
#pragma unroll
                for (int w = 0; w < kWaves; ++w) c[w] = s_w[w * Ep + tid];
#pragma unroll
                for (int w = 0; w < kWaves; ++w) { s_w[w * Ep + tid] = run; run += c[w]; }
                s_below[tid] = run;
            }
            __syncthreads();
            if (valid) {
                const int p = s_w[wave * Ep + ev] + rank;
                pos[a] = p;
                perm[p] = (int32_t)a;
            }
            __syncthreads();                        // the counters are done with
            ev = next;
        }
        return;
    }

    // ---- the tables ----
    const int e = tid;
    const int cnt = e < E ? s_total[e] : 0;
    if (blockIdx.x == 0) {
        if (e < E) counts[e] = cnt;
        // one pass of scans: offsets, the tile prefix tables of every tile height, the two size classes of every expert's rows
        int nbig = cnt / kClsBigRows, last = cnt - nbig * kClsBigRows;
        if (last > kClsSmallRows) { ++nbig; last = 0; }
        constexpr int NV = 3 + kNumTileHeights;
        int sc[NV], total[NV];
        sc[0] = cnt;
        sc[1] = e < E ? nbig : 0;
        sc[2] = e < E && last > 0 ? 1 : 0;
#pragma unroll
        for (int q = 0; q < kNumTileHeights; ++q) sc[3 + q] = e < E ? (cnt + tile_height(q) - 1) / tile_height(q) : 0;
        block_excl_scan_1024<NV>(sc, (int (*)[NV])s_wave, total, E);
        const int off = sc[0];
        if (e < E) {
            offsets[e] = off;
            cls[kClsCountsBig * (E + 1) + e] = min(cnt, nbig * kClsBigRows);
            cls[kClsCountsSmall * (E + 1) + e] = last;
            cls[kClsOffsetsSmall * (E + 1) + e] = off + nbig * kClsBigRows;
            cls[kClsPBig * (E + 1) + e] = sc[1];
            cls[kClsPSmall * (E + 1) + e] = sc[2];
#pragma unroll
            for (int q = 0; q < kNumTileHeights; ++q) tileP[q * (E + 1) + e] = sc[3 + q];
        }
        if (e == 0) {
            offsets[E] = total[0];
            cls[kClsPBig * (E + 1) + E] = total[1];
            cls[kClsPSmall * (E + 1) + E] = total[2];
#pragma unroll
            for (int q = 0; q < kNumTileHeights; ++q) tileP[q * (E + 1) + E] = total[3 + q];
        }
        return;
    }
    // Experts by descending count, ties by ascending id.  Up to 256: everybody's rank is counted, 1024 / (E rounded up to a
    // power of two) threads per expert sharing the comparisons.  More (the comparisons grow with E^2: 1000 experts
    // took 27 us of them): a bitonic sort of one key per thread.
    // Can the weight-gradient products give every XCD whole experts (expert of rank r to XCD r%8, every other
    // group of eight reversed)?  Then each operand panel is fetched by one XCD only.  Only if the reduction blocks
    // that each XCD would get stay within 10 % of the mean; the answer is control word kCtlByExpert.
    __shared__ int s_xcd[8];
    if (tid < 8) s_xcd[tid] = 0;
    int* const s_sorted = s_w;                      // counts in descending order
    if (E <= 256) {
        int* const s_rank = s_below;
        for (int i = tid; i < Ep; i += kThreads) { s_rank[i] = 0; if (i >= E) s_total[i] = -1; }   // (they never rank before an expert)
        __syncthreads();
        int width = 1;
        while (width < E) width <<= 1;
        const int me = tid & (width - 1), groups = kThreads / width;
        if (me < E) {
            const int mine = s_total[me];
            int rank = 0;
#pragma unroll 4
            for (int o = 4 * (tid / width); o < E; o += 4 * groups) {
                const int4 c = *(const int4*)&s_total[o];
                rank += (c.x > mine || (c.x == mine && o < me)) ? 1 : 0;
                rank += (c.y > mine || (c.y == mine && o + 1 < me)) ? 1 : 0;
                rank += (c.z > mine || (c.z == mine && o + 2 < me)) ? 1 : 0;
                rank += (c.w > mine || (c.w == mine && o + 3 < me)) ? 1 : 0;
            }
            if (rank) atomicAdd(&s_rank[me], rank);
        }
        __syncthreads();
        if (e < E) { order[s_rank[e]] = e; s_sorted[s_rank[e]] = cnt; }
    } else {
        unsigned long long* const s_key = (unsigned long long*)s_w;   // (kWaves * Ep ints: 1024 keys fit)
        unsigned long long key = e < E ? ((unsigned long long)(cnt + 1u) << 32) | (unsigned)(kMaxE - 1 - e) : 0ull;
        for (int k = 2; k <= kThreads; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                unsigned long long other;
                if (j < 64) other = __shfl_xor(key, j, 64);
                else {
                    __syncthreads();
                    s_key[tid] = key;
                    __syncthreads();
                    other = s_key[tid ^ j];
                }
                const bool larger = ((tid & k) == 0) == ((tid & j) == 0);   // descending: the lower thread of a pair keeps the larger key
                key = (key > other) == larger ? key : other;
            }
        }
        __syncthreads();                            // (the keys are done with)
        if (tid < E) { order[tid] = kMaxE - 1 - (int)(key & 0xffffffffu); s_sorted[tid] = (int)(key >> 32) - 1; }
    }
    __syncthreads();
    if (wave * 64 < E) {                            // ranks r and r + 16 go to one XCD, and so do r and 15 - r
        int v = tid < E ? (s_sorted[tid] + 63) / 64 : 0;
        v += __shfl_xor(v, 32, 64);
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 15, 64);
        if (lane < 8) atomicAdd(&s_xcd[lane], v);
    }
    __syncthreads();
    if (tid == 0) {
        int mx = 0, sum = 0;
        for (int x = 0; x < 8; ++x) { mx = max(mx, s_xcd[x]); sum += s_xcd[x]; }
        control[kCtlByExpert] = (E >= 8 && (long)mx * 80 <= (long)sum * 11) ? 1 : 0;
        // Strongly skewed sizes (largest expert above three times the mean): the weight-gradient products hand out
        // their tiles on demand instead of in fixed rounds; (control word kCtlSkewed).
        control[kCtlSkewed] = (E >= 2 && (long)s_sorted[0] * E > 3 * M) ? 1 : 0;
    }
}

void launch_plan(const moe_desc_t& D, const WsLayout& L, const int32_t* topk_idx, int32_t* counts,
                 int32_t* offsets, int32_t* pos, int32_t* perm, char* ws, hipStream_t st)
{
    const long M = (long)D.N * D.k;
    int32_t* hist = (int32_t*)(ws + L.hist);
    int nbits = 0;
    while ((1 << nbits) < D.E) ++nbits;
    const int chunk = (int)plan_chunk(M), Ep = (D.E + 3) & ~3;
    const bool own = M <= kOwnCounts;
    if (!own) hipLaunchKernelGGL(plan_hist, dim3(L.nb), dim3(kThreads), 0, st, topk_idx, M, D.E, chunk, hist);
    if (!allow_dynamic_lds<plan_place>((2 + kWaves) * kMaxE * (int)sizeof(int))) return;
    hipLaunchKernelGGL(plan_place, dim3(L.nb + 2), dim3(kThreads), (2 + kWaves) * Ep * sizeof(int), st, topk_idx,
                       own ? (const int32_t*)nullptr : hist, L.nb, chunk, D.E, nbits, M, counts, offsets, (int32_t*)(ws + L.tileP),
                       (int32_t*)(ws + L.order), (int32_t*)(ws + L.cls), (int32_t*)(ws + L.control), (int32_t*)(ws + L.arrive), D.E * L.arrive_cols,
                       pos, perm);
}

}  // namespace moe
