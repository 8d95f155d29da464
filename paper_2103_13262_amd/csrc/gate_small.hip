// Gate linear layer, top-k and scores for small batches (Algorithm 1: score = G(x), indices = ArgMax_k(score); Section 5.2):
// one workgroup of 1024 threads per token, everything in one launch - all E logits in fp64, the selection, the scores,
// and (for callers of them) the gate probabilities.
//
// Few tokens leave the tiled kernels one workgroup that walks the features slab by slab, a round trip to memory each, and
// take up to three launches; here all of a token's gate weights are requested at once, 16 bytes per thread and load, straight
// from W_g [d,E] as it lies in memory.  Thread i takes the 16-byte pieces i, i + T, ..., where T is the largest
// multiple of E / gcd(E, V) up to 1024 (V elements per piece): T V is then a multiple of E, so the experts of a thread's V
// elements are the same in every piece and their sums stay in V registers.  Put side by side the threads' sums are a matrix
// [T V / E][E] whose columns are then added up in a fixed tree, the same for every expert (equal gate columns give equal
// logits).  Products of two fp32-representable numbers are exact in fp64, so the selection is that of exact arithmetic up to
// fp64 summation rounding; ties go to the lower expert id.
//
// Where the line lies: every workgroup reads the whole gate matrix out of L2, so the time is that of
// ceil(N / 256) such reads by one compute unit (launch_gate_topk has the rule and its measurements).
#include <numeric>

#include "common.h"

namespace moe {
namespace {

constexpr int kThreads = 1024;
constexpr int kNone = 0x7fffffff;

template <typename T> struct Elems;
template <> struct Elems<float> {
    static constexpr int V = 4;
    static __device__ __forceinline__ void get(const uint4& p, float (&v)[4])
    {
        v[0] = __uint_as_float(p.x); v[1] = __uint_as_float(p.y); v[2] = __uint_as_float(p.z); v[3] = __uint_as_float(p.w);
    }
};
template <> struct Elems<unsigned short> {
    static constexpr int V = 8;
    static __device__ __forceinline__ void get(const uint4& p, float (&v)[8])
    {
        const unsigned w[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};

__device__ __forceinline__ bool better(double v, int i, double bv, int bi) { return v > bv || (v == bv && i < bi); }

// LDS: the threads' sums (V doubles each; the tree and the logits work in place), then the token's features as floats.
// WHOLE: E is a multiple of V, a piece lies inside one feature.  CPL: 64 CPL is at least E.  SHARED: more than 256 tokens,
// so the kernel keeps to the 64 registers with which two workgroups share a compute unit; otherwise twice as many
// pieces are on their way at a time.
template <typename T, bool WHOLE, int CPL, bool SHARED>
__global__ __launch_bounds__(kThreads, SHARED ? 8 : 4) void gate_small_kernel(const T* __restrict__ X, const T* __restrict__ Wg, const float* __restrict__ bg,
                                                              int d, int E, int k, int Tn /* threads that take part */,
                                                              int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                              double* __restrict__ probs, int rewrite, int32_t* __restrict__ fail)
{
    constexpr int V = Elems<T>::V;
    extern __shared__ __align__(16) unsigned char smem_small[];
    double* const s_sum = (double*)smem_small;                 // [Tn * V] = [rows][E]
    float* const s_x = (float*)(s_sum + kThreads * V);         // [d]
    const int tid = threadIdx.x;
    const long t = blockIdx.x;
    // the list of tokens whose every logit was evaluated in fp64: all of them
    if (fail && tid == 0) { fail[1 + t] = (int32_t)t; if (t == 0) fail[0] = (int32_t)gridDim.x; }
    for (int c = tid; c < d / V; c += kThreads) {
        float v[V];
        Elems<T>::get(((const uint4*)(X + (size_t)t * d))[c], v);
#pragma unroll
        for (int u = 0; u < V; ++u) s_x[c * V + u] = v[u];
    }
    __syncthreads();
    const int rows = Tn * V / E;                               // features between a thread's consecutive pieces
    if (tid < Tn) {
        double acc[V];
        int f[WHOLE ? 1 : V];                                  // feature of element u of the current piece
#pragma unroll
        for (int u = 0; u < V; ++u) {
            acc[u] = 0.0;
            if (!WHOLE || u == 0) f[u] = (tid * V + u) / E;
        }
        const int pieces = d * E / V;                          // (d is a multiple of 32)
        const uint4* const W = (const uint4*)Wg;
        auto add = [&](const uint4& q) {
            float w[V];
            Elems<T>::get(q, w);
#pragma unroll
            for (int u = 0; u < V; ++u) {
                acc[u] = fma((double)s_x[f[WHOLE ? 0 : u]], (double)w[u], acc[u]);
                if (!WHOLE || u == V - 1) f[WHOLE ? 0 : u] += rows;
            }
        };
        int c = tid;
        if constexpr (!SHARED) {
            constexpr int FLY = 8;                             // pieces on their way
            for (; c + (FLY - 1) * Tn < pieces; c += FLY * Tn) {
                uint4 q[FLY];
#pragma unroll
                for (int n = 0; n < FLY; ++n) q[n] = W[c + n * Tn];
#pragma unroll
                for (int n = 0; n < FLY; ++n) add(q[n]);
            }
        }
#pragma unroll 4
        for (; c < pieces; c += Tn) add(W[c]);
#pragma unroll
        for (int u = 0; u < V; ++u) s_sum[tid * V + u] = acc[u];
    }
    __syncthreads();
    // columns of [rows][E]: eight rows into one until one is left
    for (int n = rows; n > 1;) {
        const int m = (n + 7) / 8;
        for (int i = tid; i < m * E; i += kThreads) {
            double v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = i + q * m * E < n * E ? s_sum[i + q * m * E] : 0.0;
            s_sum[i] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
        __syncthreads();
        n = m;
    }
    if (tid < E) {
        double l = s_sum[tid];
        if (bg) l += (double)bg[tid];
        if (!(l == l)) l = -__builtin_inf();                   // NaN ranks last; indices stay in range
        s_sum[tid] = l;
    }
    __syncthreads();
    if (tid >= 64) return;
    // ---- selection and scores: one wavefront, a lane keeping the logits of experts lane, lane + 64, ...
    const int lane = tid;
    double l[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        l[c] = -__builtin_inf();
        if (c * 64 < E && c * 64 + lane < E) l[c] = s_sum[c * 64 + lane];
    }
    unsigned taken = 0;
    double lsel[kMaxK];
    int isel[kMaxK];
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        if (j >= k) break;
        double bv = -__builtin_inf();
        int bi = kNone;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int e = c * 64 + lane;
            if (c * 64 < E && e < E && !((taken >> c) & 1) && better(l[c], e, bv, bi)) { bv = l[c]; bi = e; }
        }
        for (int off = 32; off > 0; off >>= 1) {
            const double ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        if ((bi & 63) == lane && bi < E) taken |= 1u << (bi >> 6);
        lsel[j] = bv;
        isel[j] = bi;
    }
    double ex[kMaxK], den = 0.0;
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        if (j >= k) break;
        ex[j] = exp(lsel[j] - lsel[0]);
        den += ex[j];
    }
    if (probs) {                                               // p = softmax(l); with scores over all experts also the k scores
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            if (c * 64 < E) {
                l[c] = exp(l[c] - lsel[0]);                    // (lanes past E hold -inf: 0)
                s += l[c];
            }
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int e = c * 64 + lane;
            if (c * 64 < E && e < E) probs[(size_t)t * E + e] = l[c] / s;
        }
        if (rewrite) den = s;
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < kMaxK; ++j) {
            if (j >= k) break;
            topk_idx[t * k + j] = isel[j];
            topk_w[t * k + j] = (float)(ex[j] / den);
        }
    }
}

template <typename T, bool WHOLE, int CPL, bool SHARED>
void launch(const moe_desc_t& D, const T* X, const T* Wg, const float* bg, int32_t* topk_idx, float* topk_w, double* probs,
            int32_t* fail, hipStream_t st)
{
    constexpr int V = Elems<T>::V, kSums = kThreads * V * (int)sizeof(double);
    const int q = D.E / std::gcd(D.E, V), Tn = kThreads / q * q;
    constexpr auto kern = gate_small_kernel<T, WHOLE, CPL, SHARED>;
    if (!allow_dynamic_lds<kern>(kSums + kGateSmallMaxD * (int)sizeof(float))) return;
    hipLaunchKernelGGL(kern, dim3((unsigned)D.N), dim3(kThreads), kSums + D.d * (int)sizeof(float), st, X, Wg, bg, D.d, D.E, D.k, Tn,
                       topk_idx, topk_w, probs, D.score_all, fail);
}
template <typename T>
void launch_type(const moe_desc_t& D, const void* X, const void* Wg, const float* bg, int32_t* topk_idx, float* topk_w, double* probs,
                 int32_t* fail, hipStream_t st)
{
    const bool whole = D.E % Elems<T>::V == 0;
    auto go = [&](auto w, auto cpl) {
        constexpr int CPL = decltype(cpl)::value;
        if (CPL <= 4 && D.N > 256)
            launch<T, decltype(w)::value, CPL, CPL <= 4>(D, (const T*)X, (const T*)Wg, bg, topk_idx, topk_w, probs, fail, st);
        else launch<T, decltype(w)::value, CPL, false>(D, (const T*)X, (const T*)Wg, bg, topk_idx, topk_w, probs, fail, st);
    };
    using C4 = std::integral_constant<int, 4>;
    using C16 = std::integral_constant<int, kMaxE / 64>;
    if (D.E <= 256) { if (whole) go(std::true_type{}, C4{}); else go(std::false_type{}, C4{}); }
    else { if (whole) go(std::true_type{}, C16{}); else go(std::false_type{}, C16{}); }
}
}  // namespace

void launch_gate_small(const moe_desc_t& D, const void* X, const void* Wg, const float* bg, int32_t* topk_idx, float* topk_w,
                       double* probs, int32_t* fail, hipStream_t st)
{
    if (D.dtype == MOE_BF16) launch_type<unsigned short>(D, X, Wg, bg, topk_idx, topk_w, probs, fail, st);
    else launch_type<float>(D, X, Wg, bg, topk_idx, topk_w, probs, fail, st);
}

}  // namespace moe
