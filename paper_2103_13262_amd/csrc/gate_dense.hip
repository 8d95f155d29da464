// Gate gradient when EVERY expert receives one, for scores taken from the softmax over all experts (desc.score_all;
// Algorithm 1 with a softmax gate, Section 2.1: the gate is trained through the score).
// With p = softmax(l) and S = sum_j w_j dL/dw_j over a token's slots, an expert b outside the selection has
// dL/dl_b = -p_b S; a selected one has w_j (dL/dw_j - S).  The combine backward writes both into one dense matrix
// R[t][e] = dL/dl_e (fp32), and the gate's gradients are two small dense products of it, in one launch:
//   dWg[:, e]  = sum_t X[t][:] R[t][e],  dbg[e] = sum_t R[t][e]     by chunks of tokens (dense_final adds the chunks)
//   dX[t][:]   = sum_j dXs[pos[t,j]][:] + sum_e R[t][e] Wg[:, e]    (the expert path's rows are gathered in the epilogue)
// both on the fp32 matrix cores with 64 x 64 tiles (tile_f32.h), summed in a fixed order, every output rounded once.
// Bound by latency at few thousand tokens (a tile is 2 to 16 blocks deep), so the chunks are made as short as it takes to
// give every compute unit two tiles.  2048 tokens, d 1024, 64 experts, bf16: 126 us in five launches (vector FMA, 64
// workgroups for the weight gradient, the selected experts' terms apart) -> 27.5 us in two.
#include "common.h"
#include "tile_f32.h"

namespace moe {

namespace {
using namespace tile_f32;
typedef unsigned short u16;

constexpr int kOutPitch = TN + 4;

// part[c][e][i] and bpart[c][e] of one chunk of tokens: tile of 64 experts x 64 features, reduction over the chunk's tokens
template <typename T>
__device__ __forceinline__ void dense_dwg_tile(const T* __restrict__ X, const float* __restrict__ R, long N, int d, int E, int Ep,
                                               int chunk, int c, int i0, int e0, float* __restrict__ part,
                                               float* __restrict__ bpart, float* smem)
{
    constexpr int OP = operand_floats<true>(), BUF = 2 * OP;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const long t0 = (long)c * chunk;
    const int Kt = (int)min((long)chunk, N - t0), nblk = (Kt + TK - 1) / TK;
    Stream<true, float> sa;
    Stream<true, T> sb;
    sa.init(R + t0 * Ep + e0, Ep, Ep - e0, tid, nullptr, 0, 1);
    sb.init(X + t0 * d + i0, d, d - i0, tid, nullptr, 0, 1);
    // A block's 32 tokens are summed on their own and then added to the chunk's: a running sum over 512 tokens would round at its
    // full size 256 times (dWg of 30000 tokens in 61 experts, fp32: 1.45 times the error of sums by 64 rows of an expert).
    f32x16 sum;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.f;
    float bsum = 0.f;                    // of expert e0 + wm * 32 + lane % 32, half of the reduction indices
    float4 ra[2], rb[2];
    sa.fetch(ra, 0, Kt);
    sb.fetch(rb, 0, Kt);
    for (int b = 0; b < nblk; ++b) {
        float* const A = smem + (b & 1) * BUF;
        stash_block<true>(A, ra, tid);
        stash_block<true>(A + OP, rb, tid);
        sa.fetch(ra, b + 1, Kt - (b + 1) * TK);
        sb.fetch(rb, b + 1, Kt - (b + 1) * TK);
        __syncthreads();
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        float bacc = 0.f;
#pragma unroll
        for (int kk = 0; kk < TK / 8; ++kk) {
            float a[4], x[4];
            operand<true>(A, wm * 32, kk, lane, a);
            operand<true>(A + OP, wn * 32, kk, lane, x);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], x[s], acc, 0, 0, 0);
                bacc += a[s];
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] += acc[v];
        bsum += bacc;
    }
    const int i = i0 + wn * 32 + (lane & 31);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int e = e0 + wm * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        if (e < E && i < d) part[((size_t)c * E + e) * d + i] = sum[v];
    }
    bsum += __shfl_xor(bsum, 32, 64);
    const int eb = e0 + wm * 32 + (lane & 31);
    if (i0 == 0 && wn == 0 && lane < 32 && eb < E) bpart[(size_t)c * E + eb] = bsum;
}

// Columns of the gate matrix for rows i of dX: four consecutive experts of feature i.  (E need not be a multiple of 4.)
template <typename T> struct GateRows {
    const T* p[2];
    int k_of, E;
    __device__ __forceinline__ void init(const T* Wg, int i0, int d, int E_, int tid)
    {
        E = E_;
        k_of = (tid & 7) * 4;
#pragma unroll
        for (int q = 0; q < 2; ++q) p[q] = Wg + (size_t)min(i0 + (tid >> 3) + 32 * q, d - 1) * E;
    }
    __device__ __forceinline__ void fetch(float4 (&r)[2], int b) const
    {
        const int k = b * TK + k_of;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            r[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            if ((E & 3) == 0) { if (k < E) r[q] = load4(p[q] + k); }
            else {
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    v[u] = 0.f;
                    if (k + u < E) {
                        if constexpr (sizeof(T) == 2) v[u] = bf16_to_f32(p[q][k + u]);
                        else v[u] = p[q][k + u];
                    }
                }
                r[q] = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
};

// dX of 64 tokens x 64 features
template <typename T>
__device__ __forceinline__ void dense_dx_tile(const T* __restrict__ Wg, const float* __restrict__ R, const T* __restrict__ dXs,
                                              const int32_t* __restrict__ pos, T* __restrict__ dX, long N, int d, int E, int Ep, int k,
                                              long t0, int i0, float* smem)
{
    constexpr int OP = operand_floats<false>(), BUF = 2 * OP;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const int Mt = (int)min((long)TM, N - t0), nblk = (Ep + TK - 1) / TK;
    Stream<false, float> sa;
    GateRows<T> sb;
    sa.init(R + t0 * Ep, Ep, Mt, tid, nullptr, 0, 1);
    sb.init(Wg, i0, d, E, tid);
    // (blocks of 32 experts summed on their own, as in dense_dwg_tile: a selected expert's term is far larger than the others', which
    // would each round at its size.  dX of 2000 tokens, 1024 experts, fp32, against fp64: 6.0e-7 off with one running sum, 3.7e-7 so)
    f32x16 sum;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = 0.f;
    float4 ra[2], rb[2];
    sa.fetch(ra, 0, Ep);
    sb.fetch(rb, 0);
    for (int b = 0; b < nblk; ++b) {
        float* const A = smem + (b & 1) * BUF;
        stash_block<false>(A, ra, tid);
        stash_block<false>(A + OP, rb, tid);
        sa.fetch(ra, b + 1, Ep - (b + 1) * TK);
        sb.fetch(rb, b + 1);
        __syncthreads();
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
        for (int kk = 0; kk < TK / 8; ++kk) {
            float a[4], w[4];
            operand<false>(A, wm * 32, kk, lane, a);
            operand<false>(A + OP, wn * 32, kk, lane, w);
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], w[s], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] += acc[v];
    }
    __syncthreads();                     // the blocks are done with: their bytes take the tile, to be read row by row
#pragma unroll
    for (int v = 0; v < 16; ++v)
        smem[(wm * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3)) * kOutPitch + wn * 32 + (lane & 31)] = sum[v];
    __syncthreads();
    // thread -> 4 features of 4 tokens
    const int f = (tid & 15) * 4;
    if (i0 + f >= d) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = (tid >> 4) + 16 * q;
        if (m >= Mt) break;
        const long t = t0 + m;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int j = 0; j < k; ++j) {
            const float4 v = load4(dXs + (size_t)pos[t * k + j] * d + i0 + f);
            x.x += v.x; x.y += v.y; x.z += v.z; x.w += v.w;
        }
        const float4 g = *(const float4*)(smem + m * kOutPitch + f);
        x.x += g.x; x.y += g.y; x.z += g.z; x.w += g.w;
        T* const o = dX + (size_t)t * d + i0 + f;
        if constexpr (sizeof(T) == 2) *(uint2*)o = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
        else *(float4*)o = x;
    }
}

constexpr int kDenseSmem = 2 * 2 * (operand_floats<true>() > operand_floats<false>() ? operand_floats<true>() : operand_floats<false>());
static_assert(TM * kOutPitch <= kDenseSmem, "the output tile fits where the blocks were");

// The first ndx workgroups write dX, the others the weight gradient's chunks.  Neither reads what the other writes, unless
// the caller has dX take the place of X: then the launcher has the two follow one another.
template <typename T>
__global__ __launch_bounds__(256) void gate_dense_pair(const T* __restrict__ X, const T* __restrict__ Wg, const float* __restrict__ R,
                                                       const T* __restrict__ dXs, const int32_t* __restrict__ pos, T* __restrict__ dX,
                                                       long N, int d, int E, int Ep, int k, int ndx, int chunk,
                                                       float* __restrict__ part, float* __restrict__ bpart)
{
    __shared__ __align__(16) float smem[kDenseSmem];
    const int nti = (d + TN - 1) / TN;
    int b = blockIdx.x;
    if (b < ndx) {
        dense_dx_tile<T>(Wg, R, dXs, pos, dX, N, d, E, Ep, k, (long)(b / nti) * TM, b % nti * TN, smem);
        return;
    }
    b -= ndx;
    const int nte = (E + TM - 1) / TM;
    dense_dwg_tile<T>(X, R, N, d, E, Ep, chunk, b / (nti * nte), b % nti * TN, b / nti % nte * TM, part, bpart, smem);
}

// dWg[:, e] and dbg[e]: the chunks in ascending order, eight at a time (rounding, as in a chunk).  grid (ceil(d / 256), E)
template <typename G>
__global__ __launch_bounds__(256) void dense_final(const float* __restrict__ part, const float* __restrict__ bpart, int nch, G* __restrict__ dWg,
                                                   float* __restrict__ dbg, int d, int E, int accumulate)
{
    const int row = blockIdx.x * 256 + threadIdx.x, e = blockIdx.y;
    if (row < d) {
        float s = 0.f;
        for (int c0 = 0; c0 < nch; c0 += 8) {
            float v = 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) v += c0 + u < nch ? part[((size_t)min(c0 + u, nch - 1) * E + e) * d + row] : 0.f;
            s += v;
        }
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
        for (int c0 = 0; c0 < nch; c0 += 8) {
            float v = 0.f;
            for (int c = c0; c < min(c0 + 8, nch); ++c) v += bpart[(size_t)c * E + e];
            s += v;
        }
        dbg[e] = accumulate ? dbg[e] + s : s;
    }
}

// ---- load-balance monitor: share of the assignments and mean gate probability of every expert ----------------
// grid (chunks of kBalanceChunk tokens, ceil(E / 64)): psum[c][e] = sum of p over the chunk's tokens: 16 groups of threads
// take every 16th token, their sums are added in ascending order.  (2048 tokens, 64 experts: 158 us when a thread walked 512
// tokens and took an fp64 exponential for each -> 4.6 us, a launch's length.)
constexpr int kGroups = 16;
__global__ __launch_bounds__(kGroups * 64) void balance_partial(const double* __restrict__ p, long N, int E, double* __restrict__ psum)
{
    __shared__ double s[kGroups][64];
    const int c = blockIdx.x, lane = threadIdx.x & 63, q = threadIdx.x >> 6, e = blockIdx.y * 64 + lane;
    double v[kBalanceChunk / kGroups];
#pragma unroll
    for (int u = 0; u < kBalanceChunk / kGroups; ++u) {
        const long t = (long)c * kBalanceChunk + u * kGroups + q;
        v[u] = t < N && e < E ? p[(size_t)t * E + e] : 0.0;
    }
    double sum = 0.0;
#pragma unroll
    for (int u = 0; u < kBalanceChunk / kGroups; ++u) sum += v[u];
    s[q][lane] = sum;
    __syncthreads();
    if (q == 0 && e < E) {
#pragma unroll
        for (int g = 1; g < kGroups; ++g) sum += s[g][lane];
        psum[(size_t)c * E + e] = sum;
    }
}

// One workgroup.  Per expert 1024 / (E rounded up to a power of two) threads add every so manieth chunk, then those sums in
// ascending order; then the scalar over the experts in ascending order.
__global__ __launch_bounds__(1024) void balance_final(const double* __restrict__ psum, const int32_t* __restrict__ counts,
                                                      long N, int E, int k, int nch, float* __restrict__ fraction,
                                                      float* __restrict__ mean_prob, float* __restrict__ loss)
{
    __shared__ double s_part[1024], s_term[kMaxE];
    int width = 1;
    while (width < E) width <<= 1;
    const int e = threadIdx.x & (width - 1), q = threadIdx.x / width, nq = 1024 / width;
    double p = 0.0;
    if (e < E) {
#pragma unroll 8
        for (int c = q; c < nch; c += nq) p += psum[(size_t)c * E + e];
    }
    s_part[threadIdx.x] = p;
    __syncthreads();
    if (q == 0 && e < E) {
        // (groups past the chunks hold zeros: with two experts there are 512, 5 us of additions in a row)
        for (int g = 1; g < min(nq, nch); ++g) p += s_part[g * width + e];
        p = N > 0 ? p / (double)N : 0.0;
        const double f = N > 0 ? (double)counts[e] / ((double)N * k) : 0.0;
        if (fraction) fraction[e] = (float)f;
        if (mean_prob) mean_prob[e] = (float)p;
        s_term[e] = f * p;
    }
    __syncthreads();
    if (threadIdx.x == 0 && loss) {
        double s = 0.0;
        for (int i = 0; i < E; ++i) s += s_term[i];
        *loss = (float)(s * E);
    }
}
}  // namespace

void launch_balance_stats(const moe_desc_t& D, const WsLayout& L, const int32_t* counts, float* fraction, float* mean_prob,
                          float* loss, char* ws, hipStream_t st)
{
    double* psum = (double*)(ws + L.prob_part);
    const int nch = (D.N + kBalanceChunk - 1) / kBalanceChunk;
    if (nch > 0)
        hipLaunchKernelGGL(balance_partial, dim3((unsigned)nch, (unsigned)((D.E + 63) / 64)), dim3(kGroups * 64), 0, st,
                           (const double*)(ws + L.logits), (long)D.N, D.E, psum);
    hipLaunchKernelGGL(balance_final, dim3(1), dim3(1024), 0, st, (const double*)psum, counts, (long)D.N, D.E, D.k, nch,
                       fraction, mean_prob, loss);
}

template <typename T, typename G>
static void gate_dense_bwd(const moe_desc_t& D, const WsLayout& L, const void* X, const void* Wg, const void* dXs, const int32_t* pos,
                           void* dX, void* dWg, float* dbg, char* ws, hipStream_t st)
{
    float* part = (float*)(ws + L.dense_part);
    float* bpart = (float*)(ws + L.dense_bpart);
    const long N = D.N;
    if (N > 0) {
        const int nti = (D.d + TN - 1) / TN, nte = (D.E + TM - 1) / TM;
        const int ndx = (int)((N + TM - 1) / TM) * nti, ndw = L.dense_chunks * nti * nte;
        auto launch = [&](int blocks, int dx_blocks) {
            hipLaunchKernelGGL(gate_dense_pair<T>, dim3((unsigned)blocks), dim3(256), 0, st, (const T*)X, (const T*)Wg,
                               (const float*)(ws + L.gate_R), (const T*)dXs, pos, (T*)dX, N, D.d, D.E, gate_r_stride(D.E), D.k, dx_blocks,
                               L.dense_chunk, part, bpart);
        };
        const size_t bytes = (size_t)N * D.d * sizeof(T);
        if (overlap(X, bytes, dX, bytes)) {
            launch(ndw, 0);
            launch(ndx, ndx);
        } else launch(ndx + ndw, ndx);
    }
    hipLaunchKernelGGL(dense_final<G>, dim3((unsigned)((D.d + 255) / 256), (unsigned)D.E), dim3(256), 0, st, (const float*)part,
                       (const float*)bpart, N > 0 ? L.dense_chunks : 0, (G*)dWg, dbg, D.d, D.E, D.accumulate);
}

void launch_gate_dense_bwd(const moe_desc_t& D, const WsLayout& L, const void* X, const void* Wg, const void* dXs, const int32_t* pos,
                           void* dX, void* dWg, float* dbg, char* ws, hipStream_t st)
{
    if (D.dtype == MOE_F32) gate_dense_bwd<float, float>(D, L, X, Wg, dXs, pos, dX, dWg, dbg, ws, st);
    else if (D.grad_dtype == MOE_BF16) gate_dense_bwd<u16, u16>(D, L, X, Wg, dXs, pos, dX, dWg, dbg, ws, st);
    else gate_dense_bwd<u16, float>(D, L, X, Wg, dXs, pos, dX, dWg, dbg, ws, st);
}

}  // namespace moe
