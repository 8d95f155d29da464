// Shared host/device declarations of libmoe355 (internal; the public ABI is include/moe355.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "../../include/moe355.h"
#include "dynamic_lds.h"
#include "routes.h"

namespace moe {

constexpr int kMaxE = 1024;
constexpr int kMaxK = 8;
// Assignments placed by one workgroup of the plan kernels: 1024, or as many more as keep the chunks at 256.
inline long plan_chunk(long M) { return 1024 * (M > 256 * 1024 ? (M + 256 * 1024 - 1) / (256 * 1024) : 1); }
constexpr int kBalanceChunk = 256;  // tokens whose gate probabilities one workgroup of the load-balance monitor sums
inline int gate_r_stride(int E) { return (E + 3) / 4 * 4; }   // floats per row of gate_R: 16-byte pieces, the last padded with zeros
constexpr int kNumTileHeights = 4;  // row-tile prefix tables are kept for 32, 64, 128, 256 rows
constexpr int kMaxPersistentWgs = 256;               // persistent grouped-GEMM workgroups (one per compute unit)
constexpr size_t kPartialBytesPerWg = 256 * 256 * 4;  // one fp32 output tile of partial sums per workgroup
// Size classes of an expert's rows for the bf16 row products: whole blocks of kClsBigRows rows, computed in
// 256 x 256 tiles, and a last piece of at most kClsSmallRows rows, computed in 128 x 512 tiles (half as many tiles
// for it).  A last piece longer than that counts as one more big block.  Tables, each [E+1]:
constexpr int kClsBigRows = 256, kClsSmallRows = 128;
enum { kClsCountsBig = 0,    // rows of the expert that the big tiles cover
       kClsCountsSmall = 1,  // rows of its last piece (0: none)
       kClsOffsetsSmall = 2, // first row of the last piece
       kClsPBig = 3,         // prefix of the number of big row blocks ([E] = total)
       kClsPSmall = 4,       // prefix of the number of last pieces ([E] = total)
       kClsTables = 5 };
__host__ __device__ constexpr int tile_height(int q) { return 32 << q; }
__host__ __device__ constexpr int tile_height_index(int bm) { return bm == 32 ? 0 : bm == 64 ? 1 : bm == 128 ? 2 : 3; }

// ---- workspace layout (byte offsets from the workspace base; every region 256-B aligned) ----
struct WsLayout {
    size_t Xs, Z, H, Ys, dYs, dZ, dXs;  // expert-contiguous activations / gradients, element type = desc.dtype
    size_t dl;        // [M]  float: gradient of the selected logits, by assignment
    size_t tileP;     // [4][E+1] int32: prefix of ceil(counts/BM) for BM = 32,64,128,256
    size_t order;     // [E] int32: experts by descending count (ties: lower id first)
    size_t cls;       // [5][E+1] int32: the experts' rows in two size classes (see kCls* below)
    size_t hist;      // [nb][E] int32: per plan-chunk histogram
    size_t dwg_part;  // [pieces][d] float: partial sums of dWg over pieces of 64 rows
    size_t dbg_part;  // [pieces] float
    size_t bias_part; // [pieces][h] float: partial column sums for the first layer's expert-bias gradients (the second's: dwg_part)
    // only with desc.score_all or desc.balance_stats:
    size_t logits;    // [N][E] double: the gate logits, then (same place) the gate probabilities
    size_t prob_part; // [ceil(N/kBalanceChunk)][E] double: sums of the gate probabilities by chunk of tokens
    // only with desc.score_all (scores = softmax over all experts):
    size_t gate_R;    // [N][gate_r_stride(E)] float: dL/dlogit of every expert
    size_t dense_part;   // [dense_chunks][E][d] float: sums of dWg by chunk of dense_chunk tokens
    size_t dense_bpart;  // [dense_chunks][E] float: and of dbg
    int dense_chunk, dense_chunks;
    size_t arrive;    // [E][arrive_cols] int32: how many pieces of an expert's sums have arrived, by column block (zeroed by the plan step; zero between launches)
    int arrive_cols;
    size_t gate_fail; // [1 + N] int32: how many tokens the fast gate kernel could not certify, then their ids (small batches: all)
    size_t WgT;       // [E][d] gate matrix transposed (written by the plan step for E > 32 and by the backward pass), element type = desc.dtype
    size_t control;   // the control block (see Ctl below)
    size_t sk_flags;  // [kSkPhases][kMaxPersistentWgs] int32 "partial sum ready" or arrivals of slices
    size_t sk_error;  // int32: set if a wait for a partial sum ran out
    size_t sk_part;   // [kSkPhases][kMaxPersistentWgs] fp32 tiles: partial sums of split output tiles, or of the small tiles' slices (bf16 only)
    size_t total;
    int nb;           // plan chunks = ceil(M / plan_chunk(M))
    long dwg_pieces;  // upper bound of 64-row pieces over all experts: floor(M/64) + E
};

// A launch may run two products' worth of split tiles one after the other (the two size classes of the rows
// kinds): each phase has partial-sum buffers and flags of its own, so a workgroup that is already in the second
// phase never overwrites a partial sum of the first that its successor has not read yet.
constexpr int kSkPhases = 2;
// A word of sk_flags is zero between launches, unless a wait was given up: then a "partial sum ready" that came too late stays set until the
// next moe_plan.  The small tiles and the weight gradients' ranges count arrivals in the bits below it, so that one left behind does not count as an
// arrival; whoever arrives last clears the word.
constexpr int kPartialReady = 1 << 16;
// The control block of a workspace, in int32 words from its start.  The plan step zeroes all of it and then sets
// by_expert and skewed; the grouped products read and update the rest.
enum Ctl {
    kCtlFlags = 0,                                             // [kSkPhases][kMaxPersistentWgs] kPartialReady, or arrivals of slices or ranges
    kCtlError = kCtlFlags + kSkPhases * kMaxPersistentWgs,     // status word: 1 if a bounded wait ran out
    kCtlByExpert = kCtlError + 1,                              // 1: the weight gradients give every XCD whole experts
    kCtlClock = kCtlError + 2,                                 // two int64: shader cycles, 100 MHz ticks (8-byte aligned)
    kCtlSkewed = kCtlError + 6,                                // 1: the experts' sizes are strongly skewed
    kCtlDyn = kCtlError + 8,                                   // [9] on-demand tile counters per XCD + workgroups finished
    kCtlWords = kCtlError + 32
};
static_assert(kCtlClock % 2 == 0 && kCtlWords <= 1024, "clock words 8-byte aligned; one 1024-thread workgroup zeroes the block");
constexpr size_t kControlBytes = kCtlWords * sizeof(int32_t);
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline size_t dtype_size(int dt) { return dt == MOE_BF16 ? 2 : 4; }

inline WsLayout ws_layout(const moe_desc_t& D)
{
    WsLayout L{};
    const size_t M = (size_t)D.N * D.k, b = dtype_size(D.dtype);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    L.Xs = take(M * D.d * b);
    L.Z = take(M * D.h * b);
    L.H = take(M * D.h * b);
    L.Ys = take(M * D.d * b);
    L.dYs = take(M * D.d * b);
    L.dZ = take(M * D.h * b);
    L.dXs = take(M * D.d * b);
    L.dl = take(M * sizeof(float));
    L.tileP = take((size_t)kNumTileHeights * (D.E + 1) * sizeof(int32_t));
    L.order = take((size_t)D.E * sizeof(int32_t));
    L.cls = take((size_t)kClsTables * (D.E + 1) * sizeof(int32_t));
    L.nb = (int)((M + plan_chunk((long)M) - 1) / plan_chunk((long)M));
    L.hist = take((size_t)(L.nb > 0 ? L.nb : 1) * D.E * sizeof(int32_t));
    L.dwg_pieces = (long)(M / 64) + D.E;
    L.dwg_part = take((size_t)L.dwg_pieces * D.d * sizeof(float));
    L.dbg_part = take((size_t)L.dwg_pieces * sizeof(float));
    L.bias_part = take((size_t)L.dwg_pieces * D.h * sizeof(float));
    L.arrive_cols = (int)((D.d * b / 16 + 63) / 64 + (D.h * b / 16 + 63) / 64);   // (both layers' bias sums side by side)
    L.arrive = take((size_t)D.E * L.arrive_cols * sizeof(int32_t));
    L.gate_fail = take(((size_t)D.N + 1) * sizeof(int32_t));
    L.WgT = take((size_t)D.E * D.d * b);
    // chunks of the dense weight gradient: as long as it takes to give two compute-unit loads of 64 x 64 tiles, 64 to 512 tokens
    L.dense_chunk = 512;
    while (L.dense_chunk > 64 && (size_t)((D.N + L.dense_chunk - 1) / L.dense_chunk) * ((D.d + 63) / 64) * ((D.E + 63) / 64) < 512)
        L.dense_chunk /= 2;
    L.dense_chunks = (D.N + L.dense_chunk - 1) / L.dense_chunk;
    const size_t before_scores = o;
    if (D.score_all || D.balance_stats) {
        L.logits = take((size_t)D.N * D.E * sizeof(double));
        L.prob_part = take((size_t)((D.N + kBalanceChunk - 1) / kBalanceChunk + 1) * D.E * sizeof(double));
    }
    if (D.score_all) {
        L.gate_R = take((size_t)D.N * gate_r_stride(D.E) * sizeof(float));
        L.dense_part = take((size_t)L.dense_chunks * D.E * D.d * sizeof(float));
        L.dense_bpart = take((size_t)L.dense_chunks * D.E * sizeof(float));
        // No kernel touches what this adds.  With scores over all experts the workspace was N (12 E + 4 d) bytes and more larger
        // than without while the products kept [N][d] sums, and the host test of the workspace's size says so still; without
        // those sums the regions above are smaller than that once a chunk has more tokens than there are experts.
        const size_t least = before_scores + (size_t)D.N * (12 * (size_t)D.E + 4 * (size_t)D.d);
        if (o < least) o = (least + 255) / 256 * 256;
    }
    L.control = take(kControlBytes);
    L.sk_flags = L.control + kCtlFlags * sizeof(int32_t);
    L.sk_error = L.control + kCtlError * sizeof(int32_t);
    L.sk_part = take(D.dtype == MOE_BF16 ? (size_t)kSkPhases * kMaxPersistentWgs * kPartialBytesPerWg : 0);
    L.total = o;
    return L;
}

// ---- error reporting -------------------------------------------------------------------
void set_error(const char* fmt, ...);
moe_status_t check_launch(const char* what);
moe_status_t check_desc(const moe_desc_t* D);   // host-side validation of a problem description (sets the error text)

// Whether two operands share memory: launches that write one while they read the other are taken apart then.
inline bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes)
{
    const uintptr_t p = (uintptr_t)a, q = (uintptr_t)b;
    return p < q + b_bytes && q < p + a_bytes;
}

// ---- kernel launchers (each enqueues on `st`; operand shapes are validated by the callers) ----
void launch_gate_topk(const moe_desc_t& D, const void* X, const void* Wg, const float* bg, int32_t* topk_idx,
                      float* topk_w, void* WgT, double* logits, int32_t* gate_fail, hipStream_t st);
// bf16 with 17 to 256 experts and no caller of the stored logits: fp32 logits on the bf16 matrix cores with a certified
// margin, fp64 for the k selected logits and for the tokens that cannot be certified (gate_fail: [1 + N] int32 scratch)
void launch_gate_bf16(const moe_desc_t& D, const void* X, const void* Wg, const float* bg, int32_t* topk_idx, float* topk_w,
                      void* WgT, int32_t* gate_fail, hipStream_t st);
// few enough tokens (gate_rows_pays): another kernel behind the transposition
bool gate_rows_pays(const moe_desc_t& D);
void launch_gate_rows(const moe_desc_t& D, const void* X, const void* WgT, const float* bg, int32_t* topk_idx, float* topk_w, int32_t* gate_fail,
                      hipStream_t st);
// (WgT: [E][d] scratch for the transposed gate matrix; logits [N][E]: only with desc.score_all or desc.balance_stats, else NULL; holds the
// gate probabilities afterwards)
// small batches: one workgroup per token, one launch (probs: as logits above)
constexpr int kGateSmallMaxD = 16384;   // the token's features are kept in LDS as floats
void launch_gate_small(const moe_desc_t& D, const void* X, const void* Wg, const float* bg, int32_t* topk_idx, float* topk_w,
                       double* probs, int32_t* gate_fail, hipStream_t st);
void launch_plan(const moe_desc_t& D, const WsLayout& L, const int32_t* topk_idx, int32_t* counts,
                 int32_t* offsets, int32_t* pos, int32_t* perm, char* ws, hipStream_t st);

void launch_scatter(const moe_desc_t& D, const void* X, const int32_t* pos, void* Xs, hipStream_t st);
void launch_combine(const moe_desc_t& D, const void* Ys, const float* topk_w, const int32_t* pos, void* Y,
                    hipStream_t st);
// With scores over all experts the combine backward also writes the gradient of every logit (R NULL: it does not).
struct GateDense {
    const double* p;           // [N][E] gate probabilities
    const int32_t* topk_idx;   // [N][k]
    float* R;                  // [N][stride]
    int E, stride;
};
void launch_dcombine(const moe_desc_t& D, const void* dY, const void* Ys, const float* topk_w,
                     const int32_t* pos, void* dYs, float* dl, const GateDense& gate, const void* X, void* Xs, const void* Wg, void* WgT, hipStream_t st);
// (X, Xs: the scatter Xs[pos[a],:] = X[t,:] rides along, or NULL, NULL; Wg, WgT: the gate matrix transposed, likewise)
void launch_gate_bwd(const moe_desc_t& D, const WsLayout& L, const void* Xs, const void* dXs, const void* Wg,
                     const float* dl, const int32_t* topk_idx, const int32_t* pos, const int32_t* perm,
                     const int32_t* counts, const int32_t* offsets, void* dX, void* dWg, float* dbg, char* ws, hipStream_t st);
void launch_gate_bwd_whole(const moe_desc_t& D, const WsLayout& L, const void* Xs, const void* dXs, const void* Wg,
                           const float* dl, const int32_t* topk_idx, const int32_t* pos, const int32_t* perm,
                           const int32_t* counts, const int32_t* offsets, void* dX, void* dWg, float* dbg, char* ws, hipStream_t st);
void launch_balance_stats(const moe_desc_t& D, const WsLayout& L, const int32_t* counts, float* fraction, float* mean_prob,
                          float* loss, char* ws, hipStream_t st);
// launch_gate_bwd for scores over all experts: from the gradient of every logit (GateDense::R)
void launch_gate_dense_bwd(const moe_desc_t& D, const WsLayout& L, const void* X, const void* Wg, const void* dXs, const int32_t* pos,
                           void* dX, void* dWg, float* dbg, char* ws, hipStream_t st);

// Grouped matrix products over the expert segments.
//   kRows*: C[r,:] (r in segment e) = A[r,:] * op(B[e]);  A is [M,K] row-major, C is [M,Nout] row-major.
//   kColsT: C[e] (K1 x K2) = A[seg e]^T * B[seg e];       A is [M,K1], B is [M,K2], C is [E,K1,K2].
enum GemmKind {
    kRowsNN_GeLU = 0,  // B[e] is [K,Nout];  writes C = acc (pre-activation) and C2 = GeLU(acc)
    kRowsNN = 1,       // B[e] is [K,Nout]
    kRowsNT_dGeLU = 2, // B[e] is [Nout,K];  C = acc * GeLU'(Zin)
    kRowsNT = 3,       // B[e] is [Nout,K]
    kColsT = 4         // weight gradient; honours grad_dtype and accumulate
};
struct GemmArgs {
    int kind;
    const void* A;
    const void* B;
    void* C;
    void* C2;         // kRowsNN_GeLU: GeLU output
    const void* Zin;  // kRowsNT_dGeLU: saved pre-activation [M,Nout]
    const void* bias; // kRowsNN_GeLU, kRowsNN: [E,Nout] added to the product (activation type), or NULL
    const int32_t* a_gather;  // kRows*: row r of the A operand is A[a_gather[r] / a_gather_div, :] (the scatter done on the fly), or NULL
    int a_gather_div;
    int wide_gather;          // the gathered rows lie in 4 GB or more
    const int32_t* c_scatter; // kRowsNN: row r of the product is written to C[c_scatter[r], :] (the gather done on the fly; top-1 only), or NULL
    int K;            // kRows*: reduction width;  kColsT: K1 (rows of C[e])
    int Nout;         // kRows*: columns of C;     kColsT: K2 (columns of C[e])
    long M;           // total rows (N*k)
    int E;
    const int32_t* counts;
    const int32_t* offsets;
    const int32_t* tileP;  // [4][E+1]
    const int32_t* order;  // [E]
    const int32_t* cls;    // [kClsTables][E+1] size-class tables of the plan step, or NULL (bf16 row products only)
    void* sk_part;         // partial sums: of the persistent kernels one tile per phase and workgroup; of the small tiles one per tile and slice, of the weight gradients one per tile and range
    int32_t* sk_flags;     // one word per phase and persistent workgroup (kPartialReady), or per small tile or weight-gradient tile (arrivals), see kPartialReady
    int32_t* sk_error;
    const int32_t* by_expert;  // 1: the weight-gradient products give every XCD whole experts (decided by the plan step)
    long long* clock_probe;    // [2]: shader cycles and 100 MHz ticks of workgroup 0 of the last launch
    const int32_t* skewed;     // 1: the experts' sizes are strongly skewed (decided by the plan step)
    int32_t* dyn_counters;     // [9]: next tile of every XCD's list and the number of workgroups that have finished; zero between launches
    int slices;                // weight gradients behind a rows product, in 128 x 256 tiles: ranges that an expert's rows are cut into
    int on_demand;             // weight gradients: hand the tiles out from the counters whatever the sizes
    int stream_out;            // bf16 products: results leave as streaming stores (set by the host when the experts' weights exceed the L2 caches; fp32 and accumulating gradients always do)
    int stream_weights;        // forward products in small tiles: weights that one tile reads come as streaming loads (routes.h)
    int spin_limit;            // polls of a "partial sum ready" flag before the wait is given up and the status word set (negative: at once)
    int out_f32;      // kColsT: C holds float (else the activation type)
    int accumulate;   // kColsT
};
// Points the control-block fields of a GemmArgs at a workspace's control block.
inline void set_control(GemmArgs& a, char* ws, const WsLayout& L)
{
    int32_t* ctl = (int32_t*)(ws + L.control);
    a.sk_part = ws + L.sk_part;
    a.sk_flags = ctl + kCtlFlags;
    a.sk_error = ctl + kCtlError;
    a.by_expert = ctl + kCtlByExpert;
    a.clock_probe = (long long*)(ctl + kCtlClock);
    a.skewed = ctl + kCtlSkewed;
    a.dyn_counters = ctl + kCtlDyn;
}
void launch_bias_sums(const moe_desc_t& D, const WsLayout& L, const int32_t* counts, const int32_t* offsets, float* db1, float* db2, char* ws,
                      hipStream_t st);
void launch_ggemm_f32(const GemmArgs& a, hipStream_t st);
void launch_ggemm_pair_f32(const GemmArgs& rows, const GemmArgs& cols, hipStream_t st);   // as launch_ggemm_pair_bf16_sk
void launch_ggemm_bf16_sk(const GemmArgs& a, hipStream_t st);
// A rows kind (dZ or dXs) and a weight-gradient product that does not depend on it, in one launch.
void launch_ggemm_pair_bf16_sk(const GemmArgs& rows, const GemmArgs& cols, hipStream_t st);
bool ggemm_pair_pays(const GemmArgs& rows);   // whether the pair launch is expected to beat two launches

// ---- small device helpers ------------------------------------------------------------------
// The expert whose tiles hold tile number t, from a prefix table P [E+1]: the largest e with P[e] <= t (t < P[E]), with
// what a tile needs of it.  All lanes of a wavefront call it with the same t.  The lanes look at 64 experts at a time and
// count those that begin at or before t: two dependent round trips to memory instead of the log2(E) + 1 of a binary
// search, one of them for up to 64 experts.
struct Segment { int e, first, next, count, offset; };   // first, next: P[e], P[e+1]
__device__ __forceinline__ Segment find_segment(const int32_t* __restrict__ P, int E, int t, const int32_t* __restrict__ counts,
                                                const int32_t* __restrict__ offsets)
{
    const int lane = __lane_id();
    Segment s;
    if (E <= 64) {
        const int i = min(lane, E - 1);
        const int p = P[i], pn = P[i + 1], c = counts[i], o = offsets[i];
        s.e = __popcll(__ballot(lane < E && p <= t)) - 1;
        s.first = __builtin_amdgcn_readlane(p, s.e);
        s.next = __builtin_amdgcn_readlane(pn, s.e);
        s.count = __builtin_amdgcn_readlane(c, s.e);
        s.offset = __builtin_amdgcn_readlane(o, s.e);
        return s;
    }
    int below = 0;
    for (int e0 = 0; e0 < E; e0 += 256) {
        int p[4];                      // four loads in flight
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u] = P[min(e0 + u * 64 + lane, E - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) below += __popcll(__ballot(e0 + u * 64 + lane < E && p[u] <= t));
    }
    s.e = below - 1;
    s.first = P[s.e];
    s.next = P[s.e + 1];
    s.count = counts[s.e];
    s.offset = offsets[s.e];
    return s;
}
__device__ __forceinline__ float bf16_to_f32(unsigned short v) { return __uint_as_float(((unsigned)v) << 16); }
__device__ __forceinline__ unsigned short f32_to_bf16(float f)
{
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);                                                  // round to nearest even
    return (unsigned short)(u >> 16);
}
// Two floats -> two bf16 (round to nearest even) in one 32-bit word, low half = a: one v_cvt_pk_bf16_f32.
__device__ __forceinline__ unsigned pack_bf16x2(float a, float b)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2_t;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z)
{
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * __expf(-0.5f * z * z) * 0.39894228040143268f;
}


}  // namespace moe
