// Row-movement kernels around the expert matrix products (Section 4: "scatter" puts the
// samples of one expert into contiguous memory, "gather" puts the rows back in their original
// order; Algorithm 1: y accumulates score_i * E_i(x)), and their gradients.  All are bound by
// HBM traffic: every thread moves 16-byte pieces of a row, rows are addressed through pos/perm.
// The four movements and the plan of 32768 tokens, d 2048, 32 experts, top-2, bf16: 597 -> 551 us since scatter goes by token,
// rows are found with 32-bit divisions and the loads of a thread are issued together (2.9 TB/s of what has to move at least,
// the gate's product included; a plain copy reaches 5.1).
#include <algorithm>

#include "common.h"

namespace moe {

// 16 bytes of a row as floats: 8 bf16 or 4 fp32 elements.
template <typename T> struct Vec;
template <> struct Vec<unsigned short> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void load(const void* base, size_t chunk, float* f) { widen(((const uint4*)base)[chunk], f); }
    static __device__ __forceinline__ void widen(const uint4& v, float* f)
    {
        const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ void store(void* base, size_t chunk, const float* f)
    {
        unsigned w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = pack_bf16x2(f[2 * i], f[2 * i + 1]);
        ((uint4*)base)[chunk] = make_uint4(w[0], w[1], w[2], w[3]);
    }
};
template <> struct Vec<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void load(const void* base, size_t chunk, float* f) { widen(((const uint4*)base)[chunk], f); }
    static __device__ __forceinline__ void widen(const uint4& v, float* f)
    {
        f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
    }
    static __device__ __forceinline__ void store(void* base, size_t chunk, const float* f)
    {
        ((float4*)base)[chunk] = make_float4(f[0], f[1], f[2], f[3]);
    }
};

// Row and piece of the row of flat piece number i (cpr pieces a row).  A 64-bit division is some hundred instructions, as much as
// the rest of a piece's work; the 32-bit one, a dozen, serves every batch below 2^32 pieces (uniform over the launch).
__device__ __forceinline__ void split_piece(long i, long total, int cpr, long& t, int& c)
{
    if (total <= 0xffffffffL) {
        const unsigned q = (unsigned)i / (unsigned)cpr;
        t = q;
        c = (int)((unsigned)i - q * (unsigned)cpr);
    } else {
        t = i / cpr;
        c = (int)(i - t * cpr);
    }
}

// ---- scatter: Xs[pos[t*k+j],:] = X[t,:] ---------------------------------------------------------
// By token and not by destination row: X is read once instead of k times (Xs' rows in order ask for X's rows too far apart in
// time for a cache to hold them).
__global__ __launch_bounds__(256) void scatter_rows(const uint4* __restrict__ X, const int32_t* __restrict__ pos,
                                                    uint4* __restrict__ Xs, long N, int k, int cpr)
{
    const long total = N * cpr;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        long t;
        int c;
        split_piece(i, total, cpr, t, c);
        const uint4 x = X[i];
        for (int j = 0; j < k; ++j) Xs[(size_t)pos[t * k + j] * cpr + c] = x;
    }
}

// ---- combine: Y[t,:] = sum_j w[t,j] * Ys[pos[t*k+j], :]  (slots in ascending j, fp32) ---------
// K = k where it is 1, 2 or 4 (the loads of all slots are in flight together), 0: any k, a slot after the other.
template <typename T, int K>
__global__ __launch_bounds__(256) void combine_rows(const void* __restrict__ Ys, const float* __restrict__ topk_w,
                                                    const int32_t* __restrict__ pos, void* __restrict__ Y, long N,
                                                    int k, int cpr)
{
    constexpr int V = Vec<T>::N;
    const long total = N * cpr;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        long t;
        int c;
        split_piece(i, total, cpr, t, c);
        float acc[V];
#pragma unroll
        for (int u = 0; u < V; ++u) acc[u] = 0.f;
        if constexpr (K > 0) {
            float w[K], v[K][V];
            int p[K];
#pragma unroll
            for (int j = 0; j < K; ++j) { w[j] = topk_w[t * K + j]; p[j] = pos[t * K + j]; }
#pragma unroll
            for (int j = 0; j < K; ++j) Vec<T>::load(Ys, (size_t)p[j] * cpr + c, v[j]);
#pragma unroll
            for (int j = 0; j < K; ++j)
#pragma unroll
                for (int u = 0; u < V; ++u) acc[u] = fmaf(w[j], v[j][u], acc[u]);
        } else {
            for (int j = 0; j < k; ++j) {
                const long a = t * k + j;
                const float w = topk_w[a];
                float v[V];
                Vec<T>::load(Ys, (size_t)pos[a] * cpr + c, v);
#pragma unroll
                for (int u = 0; u < V; ++u) acc[u] = fmaf(w, v[u], acc[u]);
            }
        }
        Vec<T>::store(Y, (size_t)i, acc);
    }
}

// ---- combine backward: one wavefront per token -------------------------------------------------
//   dYs[pos[a],:] = w[a] * dY[t,:];  dw[a] = <dY[t,:], Ys[pos[a],:]>;  dl_j = w_j (dw_j - sum_i w_i dw_i)
//   (Ys == NULL: the expert outputs were not kept - top-1 with the score fixed at 1, where dl is exactly zero)
//   Rides along (X != NULL): Xs[pos[a],:] = X[t,:], the scatter that the weight gradients of the first layer and of
//   the gate read; the token's row is in hand anyway, and the backward pass saves a launch.
//   Rides along as well (WgT != NULL): WgT[e][i] = Wg[i][e], which lets the gate's part of dX read a gate column as contiguous 16-byte
//   pieces; spread over all workgroups (of which there are more than the tokens need where the matrix is large).
//   KC = k where it is 1, 2 or 4, so that no branch stands between the slots' loads; 0: any k.
template <typename T>
__device__ __forceinline__ void transpose_gate(const T* __restrict__ Wg, T* __restrict__ WgT, int d, int E, long thread, long threads)
{
    for (long i = thread; i < (long)d * E; i += threads) {
        const int e = (int)(i / d), row = (int)(i - (long)e * d);
        WgT[i] = Wg[(size_t)row * E + e];
    }
}
template <typename T, int KC>
__global__ __launch_bounds__(256) void dcombine_rows(const void* __restrict__ dY, const void* __restrict__ Ys,
                                                     const float* __restrict__ topk_w,
                                                     const int32_t* __restrict__ pos, void* __restrict__ dYs,
                                                     float* __restrict__ dl, long N, int kArg, int cpr,
                                                     const GateDense gate,   // (R NULL: only the selected logits have a gradient)
                                                     const uint4* __restrict__ X, uint4* __restrict__ Xs,
                                                     const T* __restrict__ Wg, T* __restrict__ WgT, int d, int E)
{
    if (WgT) transpose_gate(Wg, WgT, d, E, (long)blockIdx.x * 256 + threadIdx.x, (long)gridDim.x * 256);
    constexpr int V = Vec<T>::N, KM = KC > 0 ? KC : kMaxK;
    const int k = KC > 0 ? KC : kArg;
    const int lane = threadIdx.x & 63;
    const long t = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= N) return;
    float w[KM], dw[KM];
    size_t r[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        dw[j] = 0.f;
        if (j < k) { r[j] = (size_t)pos[t * k + j]; w[j] = topk_w[t * k + j]; }
    }
    for (int c = lane; c < cpr; c += 64) {
        float g[V];
        Vec<T>::load(dY, (size_t)t * cpr + c, g);
        uint4 x = make_uint4(0, 0, 0, 0);
        if (X) x = X[(size_t)t * cpr + c];
        constexpr int YN = KC > 0 ? KC : 1;       // (any k: one slot after the other, in the registers of one)
        float y[YN][V];
#pragma unroll
        for (int j = 0; j < YN; ++j)
#pragma unroll
            for (int u = 0; u < V; ++u) y[j][u] = 0.f;
        if (KC > 0 && Ys) {
#pragma unroll
            for (int j = 0; j < YN; ++j) Vec<T>::load(Ys, r[j] * cpr + c, y[j]);
        }
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            if (j >= k) break;
            if (KC == 0 && Ys) Vec<T>::load(Ys, r[j] * cpr + c, y[0]);
            float o[V];
#pragma unroll
            for (int u = 0; u < V; ++u) {
                o[u] = w[j] * g[u];
                dw[j] = fmaf(g[u], y[KC > 0 ? j : 0][u], dw[j]);
            }
            Vec<T>::store(dYs, r[j] * cpr + c, o);
            if (X) Xs[r[j] * cpr + c] = x;
        }
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        if (j >= k) break;
        float part = dw[j];
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
        dw[j] = part;
        s = fmaf(w[j], part, s);
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < KM; ++j)
            if (j < k) dl[t * k + j] = w[j] * (dw[j] - s);
    }
    if (gate.R) {      // scores over all experts: -p_e s for the experts outside the selection
        for (int e = lane; e < gate.stride; e += 64) {
            float g = e < gate.E ? (float)(-gate.p[(size_t)t * gate.E + e] * (double)s) : 0.f;
#pragma unroll
            for (int j = 0; j < KM; ++j)
                if (j < k && gate.topk_idx[t * k + j] == e) g = w[j] * (dw[j] - s);
            gate.R[(size_t)t * gate.stride + e] = g;
        }
    }
}

// ---- dX[t,:] = sum_j dXs[pos[a],:] + sum_j dl[a] * Wg[:, idx[a]] ------------------------------
// (K as for combine_rows)
template <typename T, int K, int NT>
__device__ __forceinline__ void gate_bwd_dx_body(long block, long blocks, const void* __restrict__ dXs, const void* __restrict__ WgT,
                                                 const float* __restrict__ dl, const int32_t* __restrict__ topk_idx,
                                                 const int32_t* __restrict__ pos, void* __restrict__ dX, long N, int k,
                                                 int cpr)
{
    constexpr int V = Vec<T>::N;
    const long total = N * cpr;
    for (long i = block * NT + threadIdx.x; i < total; i += blocks * NT) {
        long t;
        int c;
        split_piece(i, total, cpr, t, c);
        float acc[V];
#pragma unroll
        for (int u = 0; u < V; ++u) acc[u] = 0.f;
        if constexpr (K > 0) {
            float g[K], v[K][V], wv[K][V];
            int p[K], e[K];
#pragma unroll
            for (int j = 0; j < K; ++j) { p[j] = pos[t * K + j]; e[j] = topk_idx[t * K + j]; g[j] = dl[t * K + j]; }
#pragma unroll
            for (int j = 0; j < K; ++j) {
                Vec<T>::load(dXs, (size_t)p[j] * cpr + c, v[j]);
                Vec<T>::load(WgT, (size_t)e[j] * cpr + c, wv[j]);
            }
#pragma unroll
            for (int j = 0; j < K; ++j)
#pragma unroll
                for (int u = 0; u < V; ++u) acc[u] += v[j][u];
#pragma unroll
            for (int j = 0; j < K; ++j)
#pragma unroll
                for (int u = 0; u < V; ++u) acc[u] = fmaf(g[j], wv[j][u], acc[u]);
        } else {
            for (int j = 0; j < k; ++j) {
                float v[V];
                Vec<T>::load(dXs, (size_t)pos[t * k + j] * cpr + c, v);
#pragma unroll
                for (int u = 0; u < V; ++u) acc[u] += v[u];
            }
            for (int j = 0; j < k; ++j) {
                const long a = t * k + j;
                const float g = dl[a];
                float wv[V];
                Vec<T>::load(WgT, (size_t)topk_idx[a] * cpr + c, wv);
#pragma unroll
                for (int u = 0; u < V; ++u) acc[u] = fmaf(g, wv[u], acc[u]);
            }
        }
        Vec<T>::store(dX, (size_t)i, acc);
    }
}

// ---- dWg[:,e] = sum over rows r of segment e of dl[perm[r]] * Xs[r,:]  (fixed order) ----------
// Every expert's segment is cut into pieces of 64 rows (the 64-row tile table of the plan step), so the
// work per workgroup is the same however skewed the load is.  Each thread owns one 16-byte column piece and walks
// the rows of its piece; an expert's pieces are added in ascending order, by the last of their workgroups to arrive
// (gate_bwd_whole, segment_sums) or by a second kernel (dwg_partial's gate_bwd_tail).

// 16 bytes to where the XCDs' caches meet.  (The wait states keep the next instruction from overwriting the data registers while the
// store still reads them: the compiler sees to that for its own stores but cannot see into an assembly statement.)
__device__ __forceinline__ void store_shared(float* p, const float4 v)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    const f32x4 w = {v.x, v.y, v.z, v.w};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 2" :: "v"(p), "v"(w) : "memory");
}

// SHARED: another workgroup of the launch reads the sums (last_to_arrive, sum_pieces).  Returns the piece's segment, e = -1 past the last piece.
template <typename T, bool SHARED>
__device__ __forceinline__ Segment segment_partial(const void* __restrict__ Xs, const float* __restrict__ dl, const int32_t* __restrict__ perm,
                                                const int32_t* __restrict__ counts, const int32_t* __restrict__ offsets,
                                                const int32_t* __restrict__ P64, float* __restrict__ part, float* __restrict__ bpart, int E,
                                                int d, int cpr, int piece, int col)
{
    // 64 column threads x 8 row groups: group q walks rows 8q .. 8q+7 of the piece (all eight loads in flight); the
    // groups' sums are added in the order (((0 + 1) + 2) + ...) + 7, so the result does not depend on timing.
    constexpr int V = Vec<T>::N;
    __shared__ float s_g[64];
    __shared__ float s_acc[7][64][V];
    const int pieces = P64[E];
    Segment sg;
    if (E <= 256) {
        sg = find_segment(P64, E, piece, counts, offsets);   // (a piece past the last finds the last expert)
        if (piece >= pieces) return Segment{-1, 0, 0, 0, 0};      // uniform over the workgroup
    } else {
        // Beyond 256 experts find_segment takes several round trips, which the many pieces past the last would wait for too:
        // those leave first, and the search is one of halves over scalar loads.
        if (piece >= pieces) return Segment{-1, 0, 0, 0, 0};
        int lo = 0, hi = E;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (P64[mid] <= piece) lo = mid; else hi = mid;
        }
        sg = Segment{lo, P64[lo], P64[lo + 1], counts[lo], offsets[lo]};
    }
    const int r0 = sg.offset + (piece - sg.first) * 64;
    const int r1 = min(r0 + 64, sg.offset + sg.count);
    const int ct = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int c = col * 64 + ct;
    const bool active = c < cpr;
    // The rows are asked for before the weights, whose two dependent loads and barrier then pass under them, and are widened
    // behind the barrier (widening waits for them).  A wavefront asks for its eight rows with no branch between the loads, rows
    // past the end of the piece being its last row once more, for two where it has no more, and for none where it has
    // none: an expert with few rows has one piece with a row or two in the first wavefront.  Column sums of bf16 rows
    // 3072 wide: 100 experts with 64 rows on average 11.2 us (rows behind the weights, each under a branch of its own: 13.6; widened as
    // they arrive: 11.6); 854 experts with one row on average 20.2 us (20.8; with eight loads in every wavefront and the longer
    // search in front of the exit: 33.7).
    uint4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = make_uint4(0, 0, 0, 0);
    const uint4* const rows = (const uint4*)Xs + min(c, cpr - 1);
    const int first = __builtin_amdgcn_readfirstlane(r0 + q * 8), left = r1 - first;
    if (left > 2) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = rows[(size_t)min(first + i, r1 - 1) * cpr];
    } else if (left > 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) v[i] = rows[(size_t)min(first + i, r1 - 1) * cpr];
    }
    // (dl == nullptr: plain column sums of the segment, every row with weight 1: the expert-bias gradients)
    if (threadIdx.x < 64) s_g[threadIdx.x] = r0 + (int)threadIdx.x < r1 ? (dl ? dl[perm[r0 + threadIdx.x]] : 1.f) : 0.f;
    __syncthreads();
    float acc[V];
#pragma unroll
    for (int u = 0; u < V; ++u) acc[u] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float g = s_g[q * 8 + i];
        float x[V];
        Vec<T>::widen(v[i], x);
#pragma unroll
        for (int u = 0; u < V; ++u) acc[u] = fmaf(g, i < left ? x[u] : 0.f, acc[u]);
    }
    if (q > 0) {
#pragma unroll
        for (int u = 0; u < V; ++u) s_acc[q - 1][ct][u] = acc[u];
    }
    __syncthreads();
    if (q == 0 && active) {
#pragma unroll
        for (int g = 0; g < 7; ++g)
#pragma unroll
            for (int u = 0; u < V; ++u) acc[u] += s_acc[g][ct][u];
        float* dst = part + (size_t)piece * d + (size_t)c * V;
        if constexpr (SHARED) {
#pragma unroll
            for (int u = 0; u < V; u += 4) store_shared(dst + u, make_float4(acc[u], acc[u + 1], acc[u + 2], acc[u + 3]));
        } else {
#pragma unroll
            for (int u = 0; u < V; ++u) dst[u] = acc[u];
        }
        if (c == 0 && bpart) {
            float sdl = 0.f;
            for (int i = 0; i < 64; ++i) sdl += s_g[i];
            if constexpr (SHARED) __hip_atomic_store(bpart + piece, sdl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else bpart[piece] = sdl;
        }
    }
    return sg;
}

// The pieces' sums of one launch added up in the same launch: the workgroup that arrives last of an expert's pieces (in one column
// block) adds all of them, in ascending order whoever it is.  The sums are written and read at agent scope, where the XCDs'
// caches meet.  arrive: a counter per expert and column block, zero between launches.
__device__ __forceinline__ bool last_to_arrive(int32_t* __restrict__ arrive, int pieces)
{
    __shared__ int s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's sums have arrived ...
    __syncthreads();                                   // ... and so have those of the others
    if (threadIdx.x == 0) {
        s_last = __hip_atomic_fetch_add(arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == pieces - 1;
        if (s_last) __hip_atomic_store(arrive, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return s_last;
}
// The gate's gradients of experts without rows: zeros, written by `blocks` workgroups.  dWg holds the experts side by side, so it is walked
// element by element: whole lines where many experts in a row have none, and nothing where all have some.  (Gate backward, bf16, in a workgroup per
// column block that went from expert to expert: 100 tokens, d 2048, 1000 experts, top-2 226 us, so 16; 64 tokens, d 1024, 256 experts 58, 9; 2000
// tokens, d 2048, 256 experts, most of them without rows 78, 16.)
constexpr int kZeroElements = 4096;                    // about as many elements for a workgroup
template <typename G>
__device__ __forceinline__ void zero_empty(unsigned block, unsigned blocks, const int32_t* __restrict__ counts, G* __restrict__ dWg,
                                           float* __restrict__ dbg, int d, int E)
{
    bool some = false;
    for (int e = threadIdx.x; e < E; e += 512) some = some || counts[e] == 0;
    if (!__syncthreads_or(some)) return;
    const unsigned first = block * 512 + threadIdx.x, step = blocks * 512, skip = step % (unsigned)E;
    unsigned e = first % (unsigned)E;
#pragma unroll 4
    for (size_t i = first; i < (size_t)d * E; i += step) {
        if (counts[e] == 0) dWg[i] = 0;
        e += skip;
        if (e >= (unsigned)E) e -= E;
    }
    if (block == 0 && dbg)
        for (int q = threadIdx.x; q < E; q += 512)
            if (counts[q] == 0) dbg[q] = 0.f;
}
// Sum over pieces first .. next - 1 of part[q][c], in ascending order.
__device__ __forceinline__ float sum_pieces(const float* __restrict__ part, int first, int next, int d, int c)
{
    constexpr int FLY = 8;
    float s = 0.f;
    for (int q = first; q < next; q += FLY) {
        float f[FLY];
#pragma unroll
        for (int u = 0; u < FLY; ++u) f[u] = __hip_atomic_load(part + (size_t)min(q + u, next - 1) * d + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < FLY; ++u)
            if (q + u < next) s += f[u];
    }
    return s;
}

template <typename T>
__global__ __launch_bounds__(512) void dwg_partial(const void* __restrict__ Xs, const float* __restrict__ dl,
                                                   const int32_t* __restrict__ perm, const int32_t* __restrict__ counts,
                                                   const int32_t* __restrict__ offsets, const int32_t* __restrict__ P64,
                                                   float* __restrict__ part, float* __restrict__ bpart, int E, int d,
                                                   int cpr, const T* __restrict__ Wg, T* __restrict__ WgT)
{
    // The transposed gate matrix rides along: the kernel that follows the reduction reads it.
    const long block = ((long)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    transpose_gate(Wg, WgT, d, E, block * 512 + threadIdx.x, (long)gridDim.x * gridDim.y * gridDim.z * 512);
    // The column blocks of a piece are neighbours, so that rows of several KB are read while their pages of memory are open (gate
    // backward of 32768 tokens, d 2048, 32 experts, top-2, bf16: 149 us with a launch's pieces of the first column block in front
    // of those of the second, 137 so).  Two of them change places every four pieces: otherwise every other XCD (workgroup number
    // modulo 8) would get all the second ones, which may be mostly empty.
    const int piece = (int)(blockIdx.z * gridDim.y + blockIdx.y), col = gridDim.x == 2 ? (int)blockIdx.x ^ (piece >> 2 & 1) : (int)blockIdx.x;
    segment_partial<T, false>(Xs, dl, perm, counts, offsets, P64, part, bpart, E, d, cpr, piece, col);
}

// Plain column sums of two row matrices over the same segments (the gradients of both layers' biases), side by side in one launch:
// the column blocks of the first, then those of the second, going round from piece to piece so that an XCD (workgroup number
// modulo 8) does not get the same ones of all pieces.
// An expert's pieces are added up by the last of their workgroups; experts without rows are left to more workgroups
// behind, one for kZeroExperts experts and a column block.  With the additions in a launch of their own, and the gate's (below)
// likewise, a training step of 1000 tokens, 8 experts, d 768, h 3072, top-2 took 280 us, now 277.5.
constexpr int kZeroExperts = 16;
struct ColumnSums { const void* src; float* part; float* out; int width, cpr; };
__device__ __forceinline__ void put_sum(float* out, float s, int accumulate) { *out = accumulate ? *out + s : s; }
template <typename T>
__global__ __launch_bounds__(512) void segment_sums(ColumnSums a, ColumnSums b, const int32_t* __restrict__ counts,
                                                    const int32_t* __restrict__ offsets, const int32_t* __restrict__ P64, int E,
                                                    int32_t* __restrict__ arrive, long pieces, int accumulate)
{
    constexpr int V = Vec<T>::N;
    const long piece = (long)blockIdx.z * gridDim.y + blockIdx.y;
    const int first = (a.cpr + 63) / 64;
    const int x = (int)((blockIdx.x + (unsigned)piece) % gridDim.x);
    const ColumnSums s = x < first ? a : b;
    const int col = x < first ? x : x - first, c = col * 64 * V + (int)threadIdx.x;
    const bool mine = (int)threadIdx.x < 64 * V && c < s.width;
    if (piece >= pieces) {                          // experts without rows
        if (accumulate || piece - pieces > E / kZeroExperts) return;
        const int e0 = (int)(piece - pieces) * kZeroExperts;
        for (int e = e0; e < min(e0 + kZeroExperts, E); ++e)
            if (counts[e] == 0 && mine) s.out[(size_t)e * s.width + c] = 0.f;
        return;
    }
    const Segment sg = segment_partial<T, true>(s.src, nullptr, nullptr, counts, offsets, P64, s.part, nullptr, E, s.width, s.cpr, (int)piece, col);
    if (sg.e < 0 || !last_to_arrive(arrive + (size_t)sg.e * gridDim.x + x, sg.next - sg.first) || !mine) return;
    put_sum(s.out + (size_t)sg.e * s.width + c, sum_pieces(s.part, sg.first, sg.next, s.width, c), accumulate);
}

// grid (ceil(d / 256), E): a thread owns one row of one expert's column, so that the threads of a wavefront read
// consecutive floats of every piece; the pieces are added in ascending order (loads four at a time, sums in order).
template <typename G>
__device__ __forceinline__ void dwg_final_body(int bx, int e, const float* __restrict__ part, const float* __restrict__ bpart,
                                               const int32_t* __restrict__ P64, G* __restrict__ dWg,
                                               float* __restrict__ dbg, int d, int E, int accumulate)
{
    const int row = bx * 256 + threadIdx.x;
    const int q1 = P64[e + 1];
    if (row < d) {
        float s = 0.f;
        int q = P64[e];
        for (; q + 4 <= q1; q += 4) {
            const float a0 = part[(size_t)q * d + row], a1 = part[(size_t)(q + 1) * d + row];
            const float a2 = part[(size_t)(q + 2) * d + row], a3 = part[(size_t)(q + 3) * d + row];
            s = (((s + a0) + a1) + a2) + a3;
        }
        for (; q < q1; ++q) s += part[(size_t)q * d + row];
        const size_t i = (size_t)row * E + e;
        if constexpr (sizeof(G) == 2) {
            if (accumulate) s += bf16_to_f32(dWg[i]);
            dWg[i] = f32_to_bf16(s);
        } else {
            if (accumulate) s += dWg[i];
            dWg[i] = s;
        }
    }
    if (dbg && row == 0) {
        float s = 0.f;
        for (int q = P64[e]; q < q1; ++q) s += bpart[q];
        if (accumulate) s += dbg[e];
        dbg[e] = s;
    }
}

// The two kernels that follow the partial sums of the gate-matrix gradient, in one launch: the first fgx * E
// workgroups add every expert's pieces (dWg, dbg), the others write dX.  Neither reads what the other writes.
template <typename T, typename G, int K>
__global__ __launch_bounds__(256) void gate_bwd_tail(int fgx, const float* __restrict__ part, const float* __restrict__ bpart,
                                                     const int32_t* __restrict__ P64, G* __restrict__ dWg, float* __restrict__ dbg,
                                                     int d, int E, int accumulate, const void* __restrict__ dXs, const void* __restrict__ WgT,
                                                     const float* __restrict__ dl, const int32_t* __restrict__ topk_idx,
                                                     const int32_t* __restrict__ pos, void* __restrict__ dX, long N, int k, int cpr)
{
    const int nfinal = fgx * E;
    if ((int)blockIdx.x < nfinal)
        dwg_final_body<G>((int)blockIdx.x % fgx, (int)blockIdx.x / fgx, part, bpart, P64, dWg, dbg, d, E, accumulate);
    else
        gate_bwd_dx_body<T, K, 256>((long)blockIdx.x - nfinal, (long)gridDim.x - nfinal, dXs, WgT, dl, topk_idx, pos, dX, N, k, cpr);
}

// Gate backward in one launch, for a call that has the transposed gate matrix already: workgroups of pieces first, each expert's sums added
// up by the last of them; then `zeros` workgroups for the experts without rows; then dX.  None of these reads
// what another writes.  Bound by latency in small batches, by HBM in large ones.  A step against one whose sums are added up in a second
// launch beside dX: 256 tokens, d 64, 4 experts, fp32 42.6 -> 41.1 us; 8192 tokens and more: within what two runs differ by.
template <typename T, typename G, int K>
__global__ __launch_bounds__(512) void gate_bwd_whole(const void* __restrict__ Xs, const float* __restrict__ dl, const int32_t* __restrict__ perm,
                                                      const int32_t* __restrict__ counts, const int32_t* __restrict__ offsets,
                                                      const int32_t* __restrict__ P64, float* __restrict__ part, float* __restrict__ bpart,
                                                      int32_t* __restrict__ arrive, int pieces, int cols, int zeros, G* __restrict__ dWg, float* __restrict__ dbg,
                                                      int d, int E, int accumulate, const void* __restrict__ dXs, const void* __restrict__ WgT,
                                                      const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ pos, void* __restrict__ dX,
                                                      long N, int k, int cpr)
{
    constexpr int V = Vec<T>::N;
    const int nsum = pieces * cols, front = nsum + zeros;
    if ((int)blockIdx.x >= front) {
        gate_bwd_dx_body<T, K, 512>((long)blockIdx.x - front, (long)gridDim.x - front, dXs, WgT, dl, topk_idx, pos, dX, N, k, cpr);
        return;
    }
    if ((int)blockIdx.x >= nsum) {
        zero_empty(blockIdx.x - nsum, zeros, counts, dWg, dbg, d, E);
        return;
    }
    // (as in dwg_partial: the column blocks of a piece are neighbours, and two of them change places every four pieces)
    const int piece = (int)blockIdx.x / cols, x = (int)blockIdx.x - piece * cols, col = cols == 2 ? x ^ (piece >> 2 & 1) : x;
    const int c = col * 64 * V + (int)threadIdx.x;
    const bool mine = (int)threadIdx.x < 64 * V && c < d;
    auto put = [&](int e, float s) {
        const size_t i = (size_t)c * E + e;
        if constexpr (sizeof(G) == 2) {
            if (accumulate) s += bf16_to_f32(dWg[i]);
            dWg[i] = f32_to_bf16(s);
        } else {
            if (accumulate) s += dWg[i];
            dWg[i] = s;
        }
    };
    const Segment sg = segment_partial<T, true>(Xs, dl, perm, counts, offsets, P64, part, bpart, E, d, cpr, piece, col);
    if (sg.e < 0 || !last_to_arrive(arrive + sg.e * cols + col, sg.next - sg.first)) return;
    if (mine) put(sg.e, sum_pieces(part, sg.first, sg.next, d, c));
    if (dbg && col == 0) {                              // (uniform over the workgroup)
        __shared__ float s_b[512];
        float s = 0.f;
        for (int q = sg.first; q < sg.next; q += 512) {
            if (q + (int)threadIdx.x < sg.next) s_b[threadIdx.x] = __hip_atomic_load(bpart + q + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (threadIdx.x == 0)
                for (int i = 0; i < min(512, sg.next - q); ++i) s += s_b[i];
            __syncthreads();
        }
        if (threadIdx.x == 0) dbg[sg.e] = accumulate ? dbg[sg.e] + s : s;
    }
}

// ---- launchers -----------------------------------------------------------------------------------
static unsigned grid_for(long items)
{
    long g = (items + 255) / 256;
    if (g < 1) g = 1;
    if (g > 256 * 32) g = 256 * 32;
    return (unsigned)g;
}

// Calls f with k as a compile-time constant where the kernels have a form for it, else with 0.  k 1, 2 and 4 are the common ones;
// other k take the loop, a slot's loads behind the other's.  (Measured, not built: forms for 3 and 8 take 18 and 11 % off the
// combine backward and the gate backward on average - 16384 tokens, d 2048, bf16, k 8: 265 -> 240 and 287 -> 248 us - and 3 % off
// the combine.)
template <typename F>
static void with_k(int k, F f)
{
    if (k == 1) f(std::integral_constant<int, 1>{});
    else if (k == 2) f(std::integral_constant<int, 2>{});
    else if (k == 4) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 0>{});
}

void launch_scatter(const moe_desc_t& D, const void* X, const int32_t* pos, void* Xs, hipStream_t st)
{
    const int cpr = (int)((size_t)D.d * dtype_size(D.dtype) / 16);
    hipLaunchKernelGGL(scatter_rows, dim3(grid_for((long)D.N * cpr)), dim3(256), 0, st, (const uint4*)X, pos, (uint4*)Xs,
                       (long)D.N, D.k, cpr);
}

void launch_combine(const moe_desc_t& D, const void* Ys, const float* topk_w, const int32_t* pos, void* Y,
                    hipStream_t st)
{
    const int cpr = (int)((size_t)D.d * dtype_size(D.dtype) / 16);
    const unsigned g = grid_for((long)D.N * cpr);
    with_k(D.k, [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        if (D.dtype == MOE_BF16)
            hipLaunchKernelGGL((combine_rows<unsigned short, K>), dim3(g), dim3(256), 0, st, Ys, topk_w, pos, Y, (long)D.N, D.k, cpr);
        else
            hipLaunchKernelGGL((combine_rows<float, K>), dim3(g), dim3(256), 0, st, Ys, topk_w, pos, Y, (long)D.N, D.k, cpr);
    });
}

void launch_dcombine(const moe_desc_t& D, const void* dY, const void* Ys, const float* topk_w,
                     const int32_t* pos, void* dYs, float* dl, const GateDense& gate, const void* X, void* Xs, const void* Wg, void* WgT,
                     hipStream_t st)
{
    const int cpr = (int)((size_t)D.d * dtype_size(D.dtype) / 16);
    unsigned g = (unsigned)((D.N + 3) / 4);
    if (WgT) g = std::max(g, (unsigned)(((long)D.d * D.E + 2047) / 2048));   // (at most eight elements of the gate matrix a thread)
    with_k(D.k, [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        if (D.dtype == MOE_BF16)
            hipLaunchKernelGGL((dcombine_rows<unsigned short, K>), dim3(g), dim3(256), 0, st, dY, Ys, topk_w, pos, dYs, dl,
                               (long)D.N, D.k, cpr, gate, (const uint4*)X, (uint4*)Xs, (const unsigned short*)Wg, (unsigned short*)WgT, D.d, D.E);
        else
            hipLaunchKernelGGL((dcombine_rows<float, K>), dim3(g), dim3(256), 0, st, dY, Ys, topk_w, pos, dYs, dl, (long)D.N,
                               D.k, cpr, gate, (const uint4*)X, (uint4*)Xs, (const float*)Wg, (float*)WgT, D.d, D.E);
    });
}

// grid of dwg_partial: column blocks, then pieces (over two dimensions: one holds 65535 workgroups)
static dim3 piece_grid(long pieces, int col_blocks)
{
    const unsigned y = (unsigned)(pieces < 32768 ? pieces : 32768);
    return dim3((unsigned)col_blocks, y, (unsigned)((pieces + y - 1) / y));
}

void launch_gate_bwd(const moe_desc_t& D, const WsLayout& L, const void* Xs, const void* dXs, const void* Wg,
                     const float* dl, const int32_t* topk_idx, const int32_t* pos, const int32_t* perm,
                     const int32_t* counts, const int32_t* offsets, void* dX, void* dWg, float* dbg, char* ws, hipStream_t st)
{
    const int cpr = (int)((size_t)D.d * dtype_size(D.dtype) / 16);
    float* part = (float*)(ws + L.dwg_part);
    float* bpart = (float*)(ws + L.dbg_part);
    const int32_t* P64 = (const int32_t*)(ws + L.tileP) + tile_height_index(64) * (D.E + 1);
    const dim3 pg = piece_grid(L.dwg_pieces, (cpr + 63) / 64);
    const unsigned xg = grid_for((long)D.N * cpr);
    void* WgT = ws + L.WgT;
    const int fgx = (D.d + 255) / 256;
    const dim3 tg((unsigned)(fgx * D.E) + xg);
    auto launch = [&](auto tv, auto gv) {
        using T = decltype(tv);
        using G = decltype(gv);
        hipLaunchKernelGGL(dwg_partial<T>, pg, dim3(512), 0, st, Xs, dl, perm, counts, offsets, P64, part, bpart, D.E, D.d, cpr,
                           (const T*)Wg, (T*)WgT);
        with_k(D.k, [&](auto kc) {
            hipLaunchKernelGGL((gate_bwd_tail<T, G, decltype(kc)::value>), tg, dim3(256), 0, st, fgx, (const float*)part,
                               (const float*)bpart, P64, (G*)dWg, dbg, D.d, D.E, D.accumulate, dXs, (const void*)WgT, dl, topk_idx,
                               pos, dX, (long)D.N, D.k, cpr);
        });
    };
    if (D.dtype == MOE_F32) launch(float{}, float{});
    else if (D.grad_dtype == MOE_BF16) launch((unsigned short)0, (unsigned short)0);
    else launch((unsigned short)0, float{});
}

// launch_gate_bwd for a call whose combine backward wrote the transposed gate matrix (and whose workspace has the counters: moe_backward)
void launch_gate_bwd_whole(const moe_desc_t& D, const WsLayout& L, const void* Xs, const void* dXs, const void* Wg,
                           const float* dl, const int32_t* topk_idx, const int32_t* pos, const int32_t* perm,
                           const int32_t* counts, const int32_t* offsets, void* dX, void* dWg, float* dbg, char* ws, hipStream_t st)
{
    const int cpr = (int)((size_t)D.d * dtype_size(D.dtype) / 16), cols = (cpr + 63) / 64;
    const long dx_blocks = std::min<long>(((long)D.N * cpr + 511) / 512, 256 * 16);
    const int zeros = D.accumulate ? 0 : (int)std::min<long>(((long)D.d * D.E + kZeroElements - 1) / kZeroElements, 1024);
    const long blocks = L.dwg_pieces * cols + zeros + dx_blocks;
    if (blocks > 4 << 20) {                             // (a launch holds less than 2^32 threads)
        launch_gate_bwd(D, L, Xs, dXs, Wg, dl, topk_idx, pos, perm, counts, offsets, dX, dWg, dbg, ws, st);
        return;
    }
    const int32_t* P64 = (const int32_t*)(ws + L.tileP) + tile_height_index(64) * (D.E + 1);
    auto launch = [&](auto tv, auto gv) {
        using T = decltype(tv);
        using G = decltype(gv);
        with_k(D.k, [&](auto kc) {
            hipLaunchKernelGGL((gate_bwd_whole<T, G, decltype(kc)::value>), dim3((unsigned)blocks), dim3(512), 0, st, Xs, dl, perm, counts, offsets,
                               P64, (float*)(ws + L.dwg_part), (float*)(ws + L.dbg_part), (int32_t*)(ws + L.arrive), (int)L.dwg_pieces, cols, zeros,
                               (G*)dWg, dbg, D.d, D.E, D.accumulate, dXs, (const void*)(ws + L.WgT), topk_idx, pos, dX, (long)D.N, D.k, cpr);
        });
    };
    if (D.dtype == MOE_F32) launch(float{}, float{});
    else if (D.grad_dtype == MOE_BF16) launch((unsigned short)0, (unsigned short)0);
    else launch((unsigned short)0, float{});
}

// Column sums over every expert's segment (fixed order): db1[E][h] of dZ[M][h] and db2[E][d] of dYs[M][d], either NULL for none.
void launch_bias_sums(const moe_desc_t& D, const WsLayout& L, const int32_t* counts, const int32_t* offsets, float* db1, float* db2, char* ws,
                      hipStream_t st)
{
    auto sums = [&](size_t src, size_t part, float* out, int width) {
        return ColumnSums{ws + src, (float*)(ws + part), out, out ? width : 0, out ? (int)((size_t)width * dtype_size(D.dtype) / 16) : 0};
    };
    const ColumnSums a = sums(L.dZ, L.bias_part, db1, D.h), b = sums(L.dYs, L.dwg_part, db2, D.d);
    const int cols = (a.cpr + 63) / 64 + (b.cpr + 63) / 64;
    if (!cols) return;
    const int32_t* P64 = (const int32_t*)(ws + L.tileP) + tile_height_index(64) * (D.E + 1);
    const dim3 pg = piece_grid(L.dwg_pieces + (D.accumulate ? 0 : (D.E + kZeroExperts - 1) / kZeroExperts), cols);
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, pg, dim3(512), 0, st, a, b, counts, offsets, P64, D.E, (int32_t*)(ws + L.arrive), L.dwg_pieces, D.accumulate);
    };
    if (D.dtype == MOE_BF16) launch(segment_sums<unsigned short>);
    else launch(segment_sums<float>);
}

}  // namespace moe
