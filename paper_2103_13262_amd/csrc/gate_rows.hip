// The bf16 gate for up to some thousand tokens: logits, top-k and the softmax over the k selected logits for 17 to 256 experts, with the
// selection that of exact arithmetic, in the steps that gate_bf16.hip explains: (1) all logits in fp32 on the matrix cores together
// with a bound, (2) the candidates, (3) their logits in fp64, (4) all logits in fp64 where that does not settle a token.
//
// Few workgroups have the chip to themselves, and the time is the latency of one: so a workgroup has 16 tokens, their rows are requested all
// at once, straight into LDS, and stay there for (3) and (4), the gate matrix comes out of L2 into registers, nothing but the rows' arrival and
// the logits stands behind a barrier, and (4) is part of the kernel instead of a launch behind it.  (gate_bf16.hip stages
// 32 tokens in slabs of 64 features, a barrier each, and reads the rows a second time for (3): slower for one workgroup, but each reads the gate
// matrix for twice the tokens and more of them fit a compute unit.)
//
// The bound: a sum of n terms in ANY order is off by at most n 2^-24 S, S the sum of the terms' absolute values; a logit is the sum of KP
// parts of at most n features each, so that a term passes through at most n + KP additions.  The kernel takes four times that, and for S
// the largest value among the workgroup's tokens and experts.
#include <type_traits>

#include "common.h"

namespace moe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef unsigned short u16;

constexpr int kTok = 16;            // tokens per workgroup
constexpr int kWaves = 8;           // wavefronts per workgroup
constexpr int kTokW = kTok / kWaves; // tokens whose selection a wavefront does (32 lanes each in the fp64 part)
constexpr int kCand = 16;           // candidates per token that are told apart from the rest
constexpr float kErrFactor = 4.0f;  // safety factor on the textbook bound n 2^-24 S of an fp32 sum in any order
constexpr int kNone = 0x7fffffff;   // "no expert": loses every tie
static_assert(kCand > kMaxK && kTokW * 32 == 64, "32 lanes per token must hold the k + 1 largest");

// CG column groups of NB blocks of 16 experts, KP parts of the reduction: CG KP wavefronts.  LDS: the tokens' rows (16 x dp features, in
// 16-byte chunks; chunk c of row r lies at place c ^ r of its group of 16, so that the rows of a fragment read fall into different
// banks), the parts' fp32 logits [KP][16][16 CG NB + 1] (then the fp64 ones of eight tokens), the candidates' expert ids, the parts' largest S, and
// which tokens are left to (4).
template <int CG, int NB> struct Lds {
    static constexpr int KP = kWaves / CG, E16 = 16 * CG * NB;
    static constexpr int kLogits = (KP * kTok * (E16 + 1) * 4 + 15) / 16 * 16;
    static constexpr int kOther = kLogits + kTok * kCand * 4 + 16 * 4 + 16;
    static_assert(kLogits >= KP * kWaves * E16 * 8, "the parts' fp64 logits of a token per wavefront");
};
constexpr int kLdsBytes = 160 * 1024;
inline int padded(int d) { return (d + 127) / 128 * 128; }

__device__ __forceinline__ bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }
__device__ __forceinline__ bool better(double v, int i, double bv, int bi) { return v > bv || (v == bv && i < bi); }

__device__ __forceinline__ double wide_lo(unsigned w) { return (double)__uint_as_float(w << 16); }
__device__ __forceinline__ double wide_hi(unsigned w) { return (double)__uint_as_float(w & 0xffff0000u); }

// s[n] = sum_i x_i w[n]_i in fp64 over the 16-byte pieces c = first, first + STRIDE, ... of a token's row and NW gate rows (ascending, the
// same for every expert)
template <int NW, int STRIDE, typename Row>
__device__ __forceinline__ void dots_fp64(Row row, const u16* const (&w)[NW], int d, int first, double (&s)[NW])
{
#pragma unroll
    for (int n = 0; n < NW; ++n) s[n] = 0.0;
#pragma unroll 4
    for (int c = first; c < d / 8; c += STRIDE) {
        const u32x4 x = row(c);
        u32x4 v[NW];
#pragma unroll
        for (int n = 0; n < NW; ++n) v[n] = *(const u32x4*)(w[n] + c * 8);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double xl = wide_lo(x[q]), xh = wide_hi(x[q]);
#pragma unroll
            for (int n = 0; n < NW; ++n) {
                s[n] = fma(xl, wide_lo(v[n][q]), s[n]);
                s[n] = fma(xh, wide_hi(v[n][q]), s[n]);
            }
        }
    }
}

// The k largest of the lanes' (value, expert) pairs over groups of LANES lanes, each lane holding PER of them, and the softmax over them.
template <int PER, int LANES>
__device__ __forceinline__ void select_k(double (&v)[PER], int (&id)[PER], int k, bool write, long t, int32_t* __restrict__ topk_idx,
                                         float* __restrict__ topk_w)
{
    const int lane = threadIdx.x & 63, sub = lane % LANES, group = lane - sub;
    double l = 0.0; int e = 0;                                      // the group's lane j keeps the j-th largest
#pragma unroll 1
    for (int j = 0; j < k; ++j) {
        double bv = v[0]; int bi = id[0];
#pragma unroll
        for (int c = 1; c < PER; ++c)
            if (better(v[c], id[c], bv, bi)) { bv = v[c]; bi = id[c]; }
        for (int off = LANES / 2; off > 0; off >>= 1) {
            const double ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
#pragma unroll
        for (int c = 0; c < PER; ++c)
            if (id[c] == bi) { v[c] = -INFINITY; id[c] = kNone; }   // the owner retires the winner
        if (sub == j) { l = bv; e = bi; }
    }
    const double ex = exp(l - __shfl(l, group, 64));
    double den = 0.0;
#pragma unroll 1
    for (int j = 0; j < k; ++j) den += __shfl(ex, group + j, 64);
    if (write && sub < k) {
        topk_idx[t * k + sub] = e;
        topk_w[t * k + sub] = (float)(ex / den);
    }
}

template <int CG, int NB>
__global__ __launch_bounds__(kWaves * 64, 4) void gate_rows_kernel(const u16* __restrict__ X, const u16* __restrict__ WgT,
                                                                const float* __restrict__ bg, int N, int d, int dp, int E, int k,
                                                                int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                                int32_t* __restrict__ fail)
{
    using L = Lds<CG, NB>;
    constexpr int KP = L::KP;
    constexpr int NC = (L::E16 + 63) / 64;                          // logits per lane and token in the selection
    extern __shared__ __align__(1024) char smem[];
    char* const other = smem + kTok * dp * 2;
    float (*s_logit)[kTok][L::E16 + 1] = (float (*)[kTok][L::E16 + 1])other;
    int (*s_cand)[kCand] = (int (*)[kCand])(other + L::kLogits);
    int* s_maxabs = (int*)(other + L::kLogits + kTok * kCand * 4);  // [KP] bit patterns of the parts' largest S
    unsigned* s_left = (unsigned*)(s_maxabs + 16);                  // bit r: token r is left to (4)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = wave % CG, kp = wave / CG;
    const long t0 = (long)blockIdx.x * kTok;
    const int row_chunks = dp / 8;
    // chunk c of token row r of the workgroup
    auto token = [&](int r, int c) { return *(const u32x4*)(smem + ((size_t)r * row_chunks + (c ^ r)) * 16); };   // (r < 16: inside the group)
    {
        const unsigned base = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem);
        for (int p = wave; p < dp / 32; p += kWaves) {              // pieces of 1 KB
            const unsigned q = (unsigned)(p * 64 + lane), r = q / (unsigned)row_chunks;
            const int c = (int)(q - r * (unsigned)row_chunks) ^ (int)r;
            const u16* const src = X + (size_t)min(t0 + (long)r, (long)N - 1) * d + min(c * 8, d - 8);   // (past d: a copy that is never read)
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(base + p * 1024), "v"(src) : "memory");
        }
    }
    if (tid < KP) s_maxabs[tid] = 0;
    if (tid == 0) *s_left = 0;
    float bias_sel[NC];                                             // the biases of experts lane + 64 c, for the selection below
#pragma unroll
    for (int c = 0; c < NC; ++c) bias_sel[c] = (bg && lane + 64 * c < E) ? bg[lane + 64 * c] : 0.f;

    // ---- (1): fragments of v_mfma_f32_16x16x32_bf16: lane l holds reduction indices (l / 16) * 8 .. + 7 of row / column l % 16
    const int frow = lane & 15, fq = lane >> 4;
    constexpr unsigned kAbs = 0x7fff7fffu;
    const int steps = d / 32, s0 = kp * steps / KP, s1 = (kp + 1) * steps / KP;   // this part's 32-deep steps
    const u16* wsrc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) wsrc[b] = WgT + (size_t)min((cg * NB + b) * 16 + frow, E - 1) * d + fq * 8;   // columns past E: a copy of the last, never kept
    f32x4 acc[NB], acc_abs[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) { acc[b][v] = 0.f; acc_abs[b][v] = 0.f; }
    constexpr int FLY = 4;                                          // steps whose gate weights are on their way together
    u32x4 wv[2][FLY][NB];
    auto fetch = [&](int s, u32x4 (&w)[FLY][NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FLY; ++i) {
            const int f = min(s + i, steps - 1) * 32;
#pragma unroll
            for (int b = 0; b < NB; ++b) w[i][b] = *(const u32x4*)(wsrc[b] + f);
        }
    };
    auto multiply = [&](int s, const u32x4 (&w)[FLY][NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FLY; ++i) {
            if (s + i >= s1) break;
            const u32x4 a = token(frow, (s + i) * 4 + fq);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, w[i][b]), acc[b], 0, 0, 0);
                acc_abs[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a & kAbs), __builtin_bit_cast(bf16x8, w[i][b] & kAbs),
                                                                     acc_abs[b], 0, 0, 0);
            }
        }
    };
    fetch(s0, wv[0]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // this wavefront's pieces of the rows are there ...
    __syncthreads();                                                // ... and so are the others'
    for (int s = s0; s < s1; s += 2 * FLY) {
        fetch(s + FLY, wv[1]);
        multiply(s, wv[0]);
        fetch(s + 2 * FLY, wv[0]);
        multiply(s + FLY, wv[1]);
    }
    // accumulator element v of lane l: row (l / 16) * 4 + v, column l % 16
    {
        float sa_max = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int col = (cg * NB + b) * 16 + frow;
            float col_max = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s_logit[kp][fq * 4 + v][col] = acc[b][v];
                float sa = acc_abs[b][v];
                if (!(sa < INFINITY)) sa = INFINITY;                // (NaN or overflow: nothing can be bounded)
                col_max = fmaxf(col_max, col < E ? sa : 0.f);
            }
            if (kp == 0 && bg && col < E) col_max += fabsf(bg[col]);   // (an upper bound: the largest S of the column plus |b|)
            sa_max = fmaxf(sa_max, col_max);
            if (!(col_max < INFINITY)) sa_max = INFINITY;
        }
        for (int off = 32; off > 0; off >>= 1) sa_max = fmaxf(sa_max, __shfl_xor(sa_max, off, 64));
        if (lane == 0) atomicMax(&s_maxabs[kp], __float_as_int(sa_max));   // (non-negative floats order as their bit patterns)
    }
    __syncthreads();

    // ---- (2): wavefront w handles tokens w * kTokW .., all of them interleaved
    float band;                                                     // twice the error bound of every fp32 logit of this workgroup
    {
        float s_all = 0.f;
#pragma unroll
        for (int p = 0; p < KP; ++p) s_all += __int_as_float(s_maxabs[p]);
        const float err_unit = kErrFactor * (float)((steps + KP - 1) / KP * 32 + KP + 1) * 5.9604645e-8f;   // (n + KP + 1) 2^-24, times the safety factor
        band = 2.f * (err_unit * s_all * 1.0000005f + 1e-30f);
    }
    float cv[kTokW][NC];                                            // the fp32 logits of expert lane + 64 c
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int e = lane + 64 * c;
        const float bias = bias_sel[c];
#pragma unroll
        for (int q = 0; q < kTokW; ++q) {
            cv[q][c] = -INFINITY;
            if (e < E) {
                float l = s_logit[0][wave * kTokW + q][e];
#pragma unroll
                for (int p = 1; p < KP; ++p) l += s_logit[p][wave * kTokW + q][e];
                l += bias;
                cv[q][c] = l == l ? l : -INFINITY;                  // a NaN never wins a comparison: rank it last
            }
        }
    }
    float vk[kTokW];                                                // the k-th largest fp32 logit
    {
        unsigned taken[kTokW];
#pragma unroll
        for (int q = 0; q < kTokW; ++q) { taken[q] = 0; vk[q] = -INFINITY; }
        for (int j = 0; j < k; ++j) {
            float bv[kTokW]; int bi[kTokW];
#pragma unroll
            for (int q = 0; q < kTokW; ++q) {
                bv[q] = -INFINITY; bi[q] = kNone;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int e = lane + 64 * c;
                    if (e < E && !((taken[q] >> c) & 1) && better(cv[q][c], e, bv[q], bi[q])) { bv[q] = cv[q][c]; bi[q] = e; }
                }
            }
            for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
                for (int q = 0; q < kTokW; ++q) {
                    const float ov = __shfl_xor(bv[q], off, 64);
                    const int oi = __shfl_xor(bi[q], off, 64);
                    if (better(ov, oi, bv[q], bi[q])) { bv[q] = ov; bi[q] = oi; }
                }
            }
#pragma unroll
            for (int q = 0; q < kTokW; ++q) {
                if (bi[q] != kNone && (bi[q] & 63) == lane) taken[q] |= 1u << (bi[q] >> 6);   // the owner retires the winner
                vk[q] = bv[q];
            }
        }
    }
    // candidates: fp32 logit >= v_k - band (an expert below that is below the exact k-th largest); their ids in
    // ascending order go to s_cand.  A token is settled in (3) if the bound is finite and the candidates fit.
    int n_cand[kTokW];
#pragma unroll
    for (int q = 0; q < kTokW; ++q) {
        const int r = wave * kTokW + q;
        const float thr = vk[q] - band;
        int n = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int e = lane + 64 * c;
            const bool in = e < E && cv[q][c] >= thr;
            const unsigned long long m = __ballot(in);
            const int rank = n + __popcll(m & ((1ull << lane) - 1ull));
            if (in && rank < kCand) s_cand[r][rank] = e;
            n += __popcll(m);
        }
        n_cand[q] = band < INFINITY && n >= k && n <= kCand ? n : 0;
        if (!n_cand[q] && lane == 0 && t0 + r < N) {
            atomicOr(s_left, 1u << r);
            fail[1 + atomicAdd(fail, 1)] = (int32_t)(t0 + r);
        }
    }
    __syncthreads();                                                // (s_cand is read by other lanes than its writers)

    // ---- (3): 32 lanes per token, two candidates per pass
    {
        const int q_mine = lane >> 5, sub = lane & 31, r = wave * kTokW + q_mine;
        int n_mine = 0, n_most = 0;
#pragma unroll
        for (int q = 0; q < kTokW; ++q) {
            if (q == q_mine) n_mine = n_cand[q];
            n_most = max(n_most, n_cand[q]);
        }
        auto row = [&](int c) { return token(r, c); };
        double mine[1] = {-INFINITY}; int my_e[1] = {kNone};        // lane sub of the token's 32 holds candidate sub
        for (int j = 0; j < n_most; j += 2) {
            const int e0 = j < n_mine ? s_cand[r][j] : -1, e1 = j + 1 < n_mine ? s_cand[r][j + 1] : -1;
            const u16* const w[2] = {WgT + (size_t)max(e0, 0) * d, WgT + (size_t)max(e1, 0) * d};
            double s[2];
            dots_fp64<2, 32>(row, w, d, sub, s);
            for (int off = 16; off > 0; off >>= 1) {
                s[0] += __shfl_xor(s[0], off, 64);
                s[1] += __shfl_xor(s[1], off, 64);
            }
            if (bg) { s[0] += (double)bg[max(e0, 0)]; s[1] += (double)bg[max(e1, 0)]; }
            if (!(s[0] == s[0])) s[0] = -INFINITY;
            if (!(s[1] == s[1])) s[1] = -INFINITY;
            if (sub == j && e0 >= 0) { mine[0] = s[0]; my_e[0] = e0; }
            if (sub == j + 1 && e1 >= 0) { mine[0] = s[1]; my_e[0] = e1; }
        }
        select_k<1, 32>(mine, my_e, k, n_mine > 0 && t0 + r < N, t0 + r, topk_idx, topk_w);
    }

    // ---- (4): all logits of all 16 tokens in fp64 on the matrix cores (v_mfma_f64_16x16x4_f64; operand lane l: row / column l % 16 at depth l / 16,
    // result register v of lane l: row 4 v + l / 16, column l % 16), the parts as in (1), every expert's sum in the same order; then eight
    // tokens at a time through LDS, a wavefront each.  Such tokens come together: padding is a block of zero rows, a row that is not finite unsettles its
    // workgroup.  (1500 tokens, d 1024, 256 experts, gate_prep included: 33 us, with 16 zero rows side by side 72; one token after the other
    // 340, in gate_fix_kernel behind the slab kernel 173.  4096 tokens, d 2048, 64 experts, half of them zero: 69, 166 and 155; all logits equal 93, 189 and 267.)
    const unsigned left = *s_left;                                  // (uniform over the workgroup)
    if (left == 0) return;
    f64x4 sum[NB][2];                                               // two chains, so that a step does not wait for the one before
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) { sum[b][0][v] = 0.0; sum[b][1][v] = 0.0; }
    auto multiply64 = [&](int s, const u32x4 (&w)[FLY][NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FLY; ++i) {
            if (s + i >= s1) break;
            const u32x4 a = token(frow, (s + i) * 4 + fq);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    sum[b][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(wide_lo(a[q]), wide_lo(w[i][b][q]), sum[b][0], 0, 0, 0);
                    sum[b][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(wide_hi(a[q]), wide_hi(w[i][b][q]), sum[b][1], 0, 0, 0);
                }
        }
    };
    fetch(s0, wv[0]);
    for (int s = s0; s < s1; s += 2 * FLY) {
        fetch(s + FLY, wv[1]);
        multiply64(s, wv[0]);
        fetch(s + 2 * FLY, wv[0]);
        multiply64(s + FLY, wv[1]);
    }
    double (*const s_l64)[kWaves][L::E16] = (double (*)[kWaves][L::E16])s_logit;
#pragma unroll
    for (int half = 0; half < kTok / kWaves; ++half) {
        if (half) __syncthreads();                                  // the logits of the tokens before are done with
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 2; ++v)
                s_l64[kp][4 * v + fq][(cg * NB + b) * 16 + frow] = sum[b][0][2 * half + v] + sum[b][1][2 * half + v];
        __syncthreads();
        const int r = half * kWaves + wave;
        if (left >> r & 1) {
            double v[NC]; int id[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int e = lane + 64 * c;
                v[c] = -INFINITY; id[c] = kNone;
                if (e < E) {
                    double l = s_l64[0][wave][e];
#pragma unroll
                    for (int p = 1; p < KP; ++p) l += s_l64[p][wave][e];
                    if (bg) l += (double)bg[e];
                    v[c] = l == l ? l : -INFINITY; id[c] = e;
                }
            }
            select_k<NC, 64>(v, id, k, true, t0 + r, topk_idx, topk_w);
        }
    }
}

template <int CG, int NB>
void launch_rows(const moe_desc_t& D, const u16* X, const u16* WgT, const float* bg, int32_t* topk_idx, float* topk_w, int32_t* fail, hipStream_t st)
{
    constexpr auto kern = gate_rows_kernel<CG, NB>;
    const int dp = padded(D.d), smem = kTok * dp * 2 + Lds<CG, NB>::kOther;
    if (!allow_dynamic_lds<kern>(kLdsBytes)) return;
    hipLaunchKernelGGL(kern, dim3((unsigned)((D.N + kTok - 1) / kTok)), dim3(kWaves * 64), smem, st, X, WgT, bg, D.N, D.d, dp, D.E, D.k, topk_idx,
                       topk_w, fail);
}

}  // namespace

// Whether this kernel beats that of gate_bf16.hip.  Both sides' times (gate and plan together, top-2) of d 256 to 4096, 20 to 256 experts, 1500
// to 32768 tokens:
//   * up to a workgroup per compute unit (4096 tokens) always: 0.47 to 0.95 of the time (1500 tokens, d 1024, 32 experts 27 -> 19 us; d 2048, 64
//     experts 39 -> 28; d 256, 256 experts 27 -> 24), and the gate alone with d 32 to 224 0.67 to 1.04 (1024 to 4096 tokens, top-1, 2 and 8; above
//     1 only with 256 experts: d 128, 1024 tokens 17.8 -> 18.6);
//   * up to two with at most 64 experts and d at least 1024: 0.68 to 0.97 (8192 tokens, d 2048, 32 experts 45 -> 36; d 1024, 64 experts 32 -> 31; beyond
//     either line 0.91 to 1.5: d 512, 256 experts 35 -> 42; d 1024, 128 experts 35 -> 39);
//   * up to three with at most 32: 0.79 to 0.94 (12000 tokens, d 1024, 32 experts 36 -> 34; with 64 experts 38 -> 39).  More tokens: 0.88 to 2.2.
bool gate_rows_pays(const moe_desc_t& D)
{
    if (padded(D.d) * kTok * 2 + Lds<8, 2>::kOther > kLdsBytes) return false;   // (d above 4480)
    const int groups = (D.N + kTok - 1) / kTok;
    return groups <= 256 || (D.d >= 1024 && ((groups <= 512 && D.E <= 64) || (groups <= 768 && D.E <= 32)));
}

void launch_gate_rows(const moe_desc_t& D, const void* X, const void* WgT, const float* bg, int32_t* topk_idx, float* topk_w, int32_t* fail,
                      hipStream_t st)
{
    auto go = [&](auto cg, auto nb) { launch_rows<decltype(cg)::value, decltype(nb)::value>(D, (const u16*)X, (const u16*)WgT, bg, topk_idx, topk_w, fail, st); };
    using C1 = std::integral_constant<int, 1>;
    using C8 = std::integral_constant<int, 8>;
    if (D.E <= 32) go(std::integral_constant<int, 2>{}, C1{});
    else if (D.E <= 64) go(std::integral_constant<int, 4>{}, C1{});
    else if (D.E <= 128) go(C8{}, C1{});
    else go(C8{}, std::integral_constant<int, 2>{});
}

}  // namespace moe
