// Grouped matrix products in fp32 (used when desc.dtype is fp32): the experts' fully-connected layers applied to their
// contiguous batches (Section 3.1, the dedicated linear module; Section 4) and the matching gradients, on the fp32
// matrix cores (v_mfma_f32_32x32x2_f32: full fp32 products and sums, twice the rate of the vector unit).  One launch
// covers all experts; the tile -> expert map comes from the prefix table written by the plan step.
//
// Two forms, by the number of 64 x 64 output tiles (kFewTiles):
//   tiled    (many tiles; bound by the matrix cores): a workgroup of four wavefronts (2 x 2, each one 32 x 32 accumulator)
//            per 64 x 64 tile.  Operand blocks, 32 deep, travel through registers into two LDS buffers: block b + 2 is on its
//            way from memory while block b is multiplied and block b + 1 waits in the other buffer; one barrier per block.
//   sliced   (few tiles; bound by latency, and in the tiled form by the few compute units that get a tile): a workgroup of
//            16 wavefronts per 32 x 32 tile, each with its own slice of the reduction, operands straight from memory into
//            the matrix instructions' registers (a wavefront shares nothing, so LDS would buy nothing and a loop without
//            barriers keeps 16 wavefronts' loads in flight); the slices' sums meet in LDS, added in ascending order.
// Measured (training step; before: one 64 x 64 x 16 vector-FMA kernel per product, its loads not pipelined): N 256, d 64,
// h 128, 4 experts top-2: 172 -> 48 us (42 with the plan in one launch), a product 17-31 -> 5-6 us; N 4000, d = h = 64, 2 experts: 1672 -> 123 us; N 4096,
// d 512, h 1024, 16 experts: 1436 -> 600 us, 93 TFLOP/s in the products (the tiled form; 552 us in a kernel trace).  The line between the forms: N 500,
// d 96, h 992, 5 experts (20 tiles), second layer: 24 us with its tiles cut over four groups of a tiled workgroup, 12 us
// sliced; N 2048, d 256, h 512, 8 experts (288 tiles): 31 against 29 us; above 512 tiles every compute unit has two
// tiled workgroups to overlap and the sliced form only moves more data per product.
//
// The tiled form's staging and LDS layouts: tile_f32.h.
#include "common.h"
#include "tile_f32.h"

namespace moe {

namespace {
using namespace tile_f32;

template <int KIND> struct Kind {
    static constexpr bool A_TRANS = KIND == kColsT;                                              // A is [k][row]
    static constexpr bool B_TRANS = KIND == kRowsNN || KIND == kRowsNN_GeLU || KIND == kColsT;   // B is [k][column]
    static constexpr int BUF = operand_floats<A_TRANS>() + operand_floats<B_TRANS>();            // floats per buffer
};
template <int KIND> constexpr int tiled_bytes() { return 2 * Kind<KIND>::BUF * 4; }

// Output tile number `tile` of a product in tiles of T x T: which rows and columns, and where the operands start.
struct Tile {
    int e, Mt, Nt, Kt, n0;           // expert, valid rows / columns, reduction length, first column
    long r0;                         // rows kinds: first row in the expert-contiguous order
    const float *A, *B;              // first row (column) at reduction index 0; gathered rows: the base of A
    size_t c_off;
};
template <int KIND, int T>
__device__ __forceinline__ bool locate(const GemmArgs& g, int tile, int ntn, int ntm, Tile& t)
{
    t.n0 = tile % ntn * T;
    t.Nt = min(T, g.Nout - t.n0);
    if constexpr (KIND == kColsT) {
        t.e = tile / (ntn * ntm);
        const int m0 = (tile / ntn) % ntm * T;
        const long off = g.offsets[t.e];
        t.Kt = g.counts[t.e];
        t.Mt = min(T, g.K - m0);
        t.A = (const float*)g.A + off * g.K + m0;
        t.B = (const float*)g.B + off * g.Nout + t.n0;
        t.c_off = ((size_t)t.e * g.K + m0) * g.Nout + t.n0;
        t.r0 = 0;
    } else {
        const int32_t* P = g.tileP + tile_height_index(T) * (g.E + 1);
        const int rt = tile / ntn;
        if (rt >= P[g.E]) return false;  // (the grid is the host's upper bound; uniform over the workgroup)
        const Segment s = find_segment(P, g.E, rt, g.counts, g.offsets);
        const int m0 = (rt - s.first) * T;
        t.e = s.e;
        t.r0 = (long)s.offset + m0;
        t.Mt = min(T, s.count - m0);
        t.Kt = g.K;
        t.A = g.a_gather ? (const float*)g.A : (const float*)g.A + t.r0 * g.K;
        t.B = (const float*)g.B + (size_t)s.e * g.K * g.Nout + (Kind<KIND>::B_TRANS ? (size_t)t.n0 : (size_t)t.n0 * g.K);
        t.c_off = (size_t)t.r0 * g.Nout + t.n0;
    }
    return true;
}
__device__ __forceinline__ long source_row(const GemmArgs& g, const Tile& t, int row)
{
    return g.a_gather ? (long)(g.a_gather[t.r0 + row] / g.a_gather_div) : (long)row;
}
// Writes element (m, n) of a tile: acc is its sum.
template <int KIND>
__device__ __forceinline__ void store_element(const GemmArgs& g, const Tile& t, int m, int n, float acc)
{
    float* const C = (float*)g.C;
    const size_t o = t.c_off + (size_t)m * g.Nout + n;
    float x = acc;
    if constexpr (KIND == kRowsNN || KIND == kRowsNN_GeLU) {
        if (g.bias) x += ((const float*)g.bias)[(size_t)t.e * g.Nout + t.n0 + n];
    }
    if constexpr (KIND == kRowsNN_GeLU) { C[o] = x; ((float*)g.C2)[o] = gelu_f(x); }
    else if constexpr (KIND == kRowsNT_dGeLU) C[o] = x * gelu_grad_f(((const float*)g.Zin)[o]);
    else if constexpr (KIND == kColsT) C[o] = g.accumulate ? C[o] + x : x;
    else if constexpr (KIND == kRowsNN) {          // (top-1: the row goes straight to its token's place in Y)
        if (g.c_scatter) C[(size_t)g.c_scatter[t.r0 + m] * g.Nout + t.n0 + n] = x;
        else C[o] = x;
    } else C[o] = x;
}

template <int KIND>
__device__ __forceinline__ void tiled_product(const GemmArgs& g, int tile, int ntn, int ntm, float* smem)
{
    using K = Kind<KIND>;
    const int lane = threadIdx.x & 63, tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    Tile t;
    if (!locate<KIND, TM>(g, tile, ntn, ntm, t)) return;
    Stream<K::A_TRANS, float> sa;
    Stream<K::B_TRANS, float> sb;
    sa.init(t.A, g.K, t.Mt, tid, KIND == kColsT ? nullptr : g.a_gather, t.r0, g.a_gather_div);
    sb.init(t.B, K::B_TRANS ? g.Nout : g.K, t.Nt, tid, nullptr, 0, 1);
    const int nblk = (t.Kt + TK - 1) / TK;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    float4 ra[2][2], rb[2][2];           // blocks on their way, by parity
    auto fetch = [&](int b, auto par) {
        constexpr int p = decltype(par)::value;
        sa.fetch(ra[p], b, t.Kt - b * TK);
        sb.fetch(rb[p], b, t.Kt - b * TK);
    };
    auto stash = [&](auto par) {
        constexpr int p = decltype(par)::value;
        stash_block<K::A_TRANS>(smem + p * K::BUF, ra[p], tid);
        stash_block<K::B_TRANS>(smem + p * K::BUF + operand_floats<K::A_TRANS>(), rb[p], tid);
    };
    auto multiply = [&](auto par) {
        const float* A = smem + decltype(par)::value * K::BUF;
        const float* B = A + operand_floats<K::A_TRANS>();
#pragma unroll
        for (int kk = 0; kk < TK / 8; ++kk) {
            float a[4], b[4];
            operand<K::A_TRANS>(A, wm * 32, kk, lane, a);
            operand<K::B_TRANS>(B, wn * 32, kk, lane, b);
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], b[s], acc, 0, 0, 0);
        }
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    if (nblk > 0) {
        fetch(0, even);
        fetch(1, odd);
        for (int b = 0; b < nblk; b += 2) {
            stash(even);
            fetch(b + 2, even);
            __syncthreads();
            multiply(even);
            if (b + 1 < nblk) {
                stash(odd);
                fetch(b + 3, odd);
                __syncthreads();
                multiply(odd);
            }
        }
    }
    // accumulator element v of lane l: row (v / 4) * 8 + (l / 32) * 4 + v % 4, column l % 32 of the wavefront's 32 x 32
    const int n = wn * 32 + (lane & 31);
    if (n >= t.Nt) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = wm * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        if (m < t.Mt) store_element<KIND>(g, t, m, n, acc[v]);
    }
}

constexpr int SW = 16, ST = 32;          // wavefronts (slices of the reduction) of a workgroup, tile edge
constexpr int kSlicedBytes = SW * ST * ST * 4;

// A wavefront's 16-byte (reduction index fastest) or 4-byte loads of a chunk of 16 reduction indices: lane l gets
// indices 8 kk + 4 (l / 32) .. + 3, kk = 0, 1, of row / column l % 32.
template <bool TRANS>
__device__ __forceinline__ void load_chunk(const float* p, long ld, int k0, int k_end, int lane, float (&v)[2][4])
{
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int k = k0 + kk * 8 + (lane >> 5) * 4;
        if constexpr (!TRANS) {          // (the reduction length is a multiple of 32: a chunk exists as a whole or not at all)
            float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k < k_end) q = *(const float4*)(p + k);
            v[kk][0] = q.x; v[kk][1] = q.y; v[kk][2] = q.z; v[kk][3] = q.w;
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) v[kk][s] = k + s < k_end ? p[(long)(k + s) * ld] : 0.f;
        }
    }
}

template <int KIND>
__device__ __forceinline__ void sliced_product(const GemmArgs& g, int tile, int ntn, int ntm, float* smem)
{
    using K = Kind<KIND>;
    const int lane = threadIdx.x & 63, rc = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Tile t;
    if (!locate<KIND, ST>(g, tile, ntn, ntm, t)) return;
    const int row = min(rc, t.Mt - 1), col = min(rc, t.Nt - 1);
    const float* pa = K::A_TRANS ? t.A + row : t.A + source_row(g, t, row) * g.K;
    const float* pb = K::B_TRANS ? t.B + col : t.B + (long)col * g.K;
    // slice: 16-deep chunks [c0, c1)
    const int nch = (t.Kt + 15) / 16, per = (nch + SW - 1) / SW, c0 = min(wave * per, nch), c1 = min(c0 + per, nch);
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    float a[2][2][4], b[2][2][4];        // chunks by parity
    auto fetch = [&](int c, auto par) {
        constexpr int p = decltype(par)::value;
        const int k_end = c < c1 ? t.Kt : 0;
        load_chunk<K::A_TRANS>(pa, g.K, c * 16, k_end, lane, a[p]);
        load_chunk<K::B_TRANS>(pb, g.Nout, c * 16, k_end, lane, b[p]);
    };
    auto multiply = [&](auto par) {
        constexpr int p = decltype(par)::value;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[p][kk][s], b[p][kk][s], acc, 0, 0, 0);
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    if (c0 < c1) {
        fetch(c0, even);
        fetch(c0 + 1, odd);
        for (int c = c0; c < c1; c += 2) {
            multiply(even);
            fetch(c + 2, even);
            multiply(odd);               // (past the slice's end: zeros)
            fetch(c + 3, odd);
        }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) smem[wave * (ST * ST) + ((v >> 2) * 8 + (lane >> 5) * 4 + (v & 3)) * ST + rc] = acc[v];
    __syncthreads();
    const int m = threadIdx.x >> 5, n = threadIdx.x & 31;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < SW; ++w) sum += smem[w * (ST * ST) + threadIdx.x];
    if (m < t.Mt && n < t.Nt) store_element<KIND>(g, t, m, n, sum);
}

template <int KIND>
__global__ __launch_bounds__(256) void ggemm_f32_tiled(GemmArgs g, int ntn, int ntm)
{
    __shared__ __align__(16) float smem[tiled_bytes<KIND>() / 4];
    tiled_product<KIND>(g, blockIdx.x, ntn, ntm, smem);
}
template <int KIND>
__global__ __launch_bounds__(SW * 64) void ggemm_f32_sliced(GemmArgs g, int ntn, int ntm)
{
    __shared__ __align__(16) float smem[kSlicedBytes / 4];
    sliced_product<KIND>(g, blockIdx.x, ntn, ntm, smem);
}
// A rows kind and the weight gradient that does not depend on it, in one launch: the first n1 workgroups take the tiles
// of the first, the others those of the second.
template <int KIND>
__global__ __launch_bounds__(256) void ggemm_f32_pair_tiled(GemmArgs g1, int ntn1, int n1, GemmArgs g2, int ntn2, int ntm2)
{
    constexpr int s1 = tiled_bytes<KIND>(), s2 = tiled_bytes<kColsT>();
    __shared__ __align__(16) float smem[(s1 > s2 ? s1 : s2) / 4];
    if ((int)blockIdx.x < n1) tiled_product<KIND>(g1, blockIdx.x, ntn1, 0, smem);
    else tiled_product<kColsT>(g2, (int)blockIdx.x - n1, ntn2, ntm2, smem);
}
template <int KIND>
__global__ __launch_bounds__(SW * 64) void ggemm_f32_pair_sliced(GemmArgs g1, int ntn1, int n1, GemmArgs g2, int ntn2, int ntm2)
{
    __shared__ __align__(16) float smem[kSlicedBytes / 4];
    if ((int)blockIdx.x < n1) sliced_product<KIND>(g1, blockIdx.x, ntn1, 0, smem);
    else sliced_product<kColsT>(g2, (int)blockIdx.x - n1, ntn2, ntm2, smem);
}

struct Grid { int ntn, ntm; long tiles; };
Grid grid_of(const GemmArgs& a, int T)
{
    Grid q{(a.Nout + T - 1) / T, (a.K + T - 1) / T, 0};
    // rows kinds: sum_e ceil(c_e / T) <= floor(M / T) + E
    q.tiles = a.kind == kColsT ? (long)q.ntn * q.ntm * a.E : (a.M / T + a.E) * q.ntn;
    return q;
}
constexpr long kFewTiles = 512;   // two 64 x 64 tiles per compute unit

template <int KIND> void launch_kind(const GemmArgs& a, hipStream_t st)
{
    const Grid q = grid_of(a, TM);
    if (q.tiles > kFewTiles) {
        hipLaunchKernelGGL((ggemm_f32_tiled<KIND>), dim3((unsigned)q.tiles), dim3(256), 0, st, a, q.ntn, q.ntm);
        return;
    }
    const Grid s = grid_of(a, ST);
    hipLaunchKernelGGL((ggemm_f32_sliced<KIND>), dim3((unsigned)s.tiles), dim3(SW * 64), 0, st, a, s.ntn, s.ntm);
}
template <int KIND> void launch_pair_kind(const GemmArgs& r, const GemmArgs& c, hipStream_t st)
{
    const Grid qr = grid_of(r, TM), qc = grid_of(c, TM);
    if (qr.tiles + qc.tiles > kFewTiles) {
        hipLaunchKernelGGL((ggemm_f32_pair_tiled<KIND>), dim3((unsigned)(qr.tiles + qc.tiles)), dim3(256), 0, st, r, qr.ntn,
                           (int)qr.tiles, c, qc.ntn, qc.ntm);
        return;
    }
    const Grid sr = grid_of(r, ST), sc = grid_of(c, ST);
    hipLaunchKernelGGL((ggemm_f32_pair_sliced<KIND>), dim3((unsigned)(sr.tiles + sc.tiles)), dim3(SW * 64), 0, st, r, sr.ntn,
                       (int)sr.tiles, c, sc.ntn, sc.ntm);
}
}  // namespace

void launch_ggemm_f32(const GemmArgs& a, hipStream_t st)
{
    switch (a.kind) {
        case kRowsNN_GeLU: launch_kind<kRowsNN_GeLU>(a, st); break;
        case kRowsNN: launch_kind<kRowsNN>(a, st); break;
        case kRowsNT_dGeLU: launch_kind<kRowsNT_dGeLU>(a, st); break;
        case kRowsNT: launch_kind<kRowsNT>(a, st); break;
        default: launch_kind<kColsT>(a, st); break;
    }
}

void launch_ggemm_pair_f32(const GemmArgs& rows, const GemmArgs& cols, hipStream_t st)
{
    if (rows.kind == kRowsNT_dGeLU) launch_pair_kind<kRowsNT_dGeLU>(rows, cols, st);
    else launch_pair_kind<kRowsNT>(rows, cols, st);
}

}  // namespace moe
