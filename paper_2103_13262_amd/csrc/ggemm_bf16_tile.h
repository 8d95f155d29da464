// Grouped bf16 matrix products with few rows per expert: a workgroup of four wavefronts per output tile (or per slice of its
// reduction), several workgroups on a compute unit.
//
// With up to a hundred rows per expert a row product is a stream of weights: every expert's matrix is read once for a few
// rows, and the time is the memory's as long as enough of it is on its way at any moment.  So the tiles are narrow (128 columns)
// and the workgroups small (rings of two slots, 40 to 64 KB): two to four of them on a compute unit hide each other's first loads, barriers and
// epilogues, which cost a persistent workgroup with a 256-wide tile 8 to 10 us per launch, and the hardware hands the tiles out.
//
// A tile is BM rows x 128 columns; each wavefront computes 32 columns of all rows (BM 128: 64 of 64 rows) with
// v_mfma_f32_32x32x16_bf16.  The weights are the instruction's first operand, so a lane holds four consecutive columns of one row
// and, after one exchange between the wavefront's halves, eight.
// Where the tiles are too few to fill the chip, the reduction is cut into S slices (the host chooses S from the largest possible number
// of tiles): every slice but the last to finish leaves its sum in fp32, and the last one adds them in ascending order, its own among
// them, so results do not depend on the timing, and nobody waits.
#pragma once
#include <algorithm>

#include "bf16_tiles.h"
#include "gauss.h"

namespace moe {
namespace sk {

constexpr int kTileDepth = 64;    // reduction indices of a block

template <int KIND, int BM_, int STAGES_> struct TileCfg {
    static constexpr int BM = BM_, BN = kTileCols, BK = kTileDepth, NW = 4, NT = 256, STAGES = STAGES_;
    static constexpr int WM = BM >= 128 ? 2 : 1, WN = NW / WM, TM = BM / 32 / WM, TN = BN / 32 / WN;   // wavefronts, and 32 x 32 blocks of each
    static constexpr bool B_TRANS = KIND == kRowsNN || KIND == kRowsNN_GeLU;
    static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int LA = A_BYTES / 1024 / NW, LB = B_BYTES / 1024 / NW, PER = LA + LB;
    static constexpr bool DGELU = KIND == kRowsNT_dGeLU;  // results wait in LDS in fp32 for the saved pre-activations
    static constexpr int PITCH = BN * (DGELU ? 4 : 2) + 16;   // bytes of a row of results in LDS
    static constexpr int RESULTS = BM * PITCH * (KIND == kRowsNN_GeLU ? 2 : 1);
    static constexpr int SMEM = std::max(STAGES * STAGE_BYTES, RESULTS);
};

template <int KIND, int BM, int STAGES, int OCC>
__global__ __launch_bounds__(256, OCC) void ggemm_tile_kernel(GemmArgs g, int ntn, int slices)
{
    using C = TileCfg<KIND, BM, STAGES>;
    constexpr int BK = C::BK, TM = C::TM, TN = C::TN, PER = C::PER, KS = BK / 16;
    extern __shared__ __align__(1024) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- which tile: every XCD takes a contiguous share; inside an expert the row blocks run fastest, so that those which read
    // the same weights run side by side on one XCD, then the slices, then the columns
    const int32_t* P = g.tileP + tile_height_index(BM) * (g.E + 1);
    const long per_row_tile = (long)ntn * slices;
    const int xcd = blockIdx.x & 7;
    const long idx = blockIdx.x >> 3;
    Segment sg;
    long L;
    auto place = [&](int row_tiles) {      // this workgroup's number among all tiles' slices, or -1: nothing left for it
        const long T = (long)row_tiles * per_row_tile, share = T >> 3;
        const int extra = (int)(T & 7);
        return idx < share + (xcd < extra ? 1 : 0) ? xcd * share + min(xcd, extra) + idx : -1L;
    };
    if (g.E <= 64) {                       // all that is needed of the tables in one round trip: a lane per expert
        const int i = min(lane, g.E - 1);
        const int p = P[i], pn = P[i + 1], c = g.counts[i], o = g.offsets[i];
        L = place(__builtin_amdgcn_readlane(pn, g.E - 1));
        if (L < 0) return;
        sg.e = __popcll(__ballot(lane < g.E && (long)p * per_row_tile <= L)) - 1;
        sg.first = __builtin_amdgcn_readlane(p, sg.e);  sg.next = __builtin_amdgcn_readlane(pn, sg.e);
        sg.count = __builtin_amdgcn_readlane(c, sg.e);  sg.offset = __builtin_amdgcn_readlane(o, sg.e);
    } else {
        L = place(P[g.E]);
        if (L < 0) return;
        sg = find_segment(P, g.E, (int)(L / per_row_tile), g.counts, g.offsets);
    }
    const int e = __builtin_amdgcn_readfirstlane(sg.e), mte = __builtin_amdgcn_readfirstlane(sg.next - sg.first);
    const int local = __builtin_amdgcn_readfirstlane((int)(L - (long)sg.first * per_row_tile));
    const int mt = local % mte, slice = local / mte % slices, nt = local / mte / slices;
    const int Mt = min(BM, __builtin_amdgcn_readfirstlane(sg.count) - mt * BM), n0 = nt * C::BN, Nt = min(C::BN, g.Nout - n0);
    const long row0 = (long)__builtin_amdgcn_readfirstlane(sg.offset) + (long)mt * BM;
    const int nkT = (g.K + BK - 1) / BK;
    const int kb0 = (int)((long)slice * nkT / slices), kb1 = (int)((long)(slice + 1) * nkT / slices), nk = kb1 - kb0;   // (at least one block: host)
    const int rem = min(BK, g.K - (kb1 - 1) * BK);      // (a multiple of 32)

    // ---- streams
    const bool streaming = g.stream_out;
    unsigned va[C::LA], vb[C::LB];
    setup_offsets<false, BM, 4, C::LA, BK>(g.K, Mt, wave, lane, va, g.a_gather, row0, g.a_gather_div);
    const long ldb = C::B_TRANS ? g.Nout : g.K;
    setup_offsets<C::B_TRANS, C::BN, 4, C::LB, BK>(ldb, Nt, wave, lane, vb);
    const long stepB = C::B_TRANS ? (long)BK * ldb : BK;
    const u16* qa = scalar((const u16*)g.A + (g.a_gather ? 0 : row0 * g.K) + (long)kb0 * BK);
    const u16* qb = scalar((const u16*)g.B + (size_t)e * g.K * g.Nout + (C::B_TRANS ? (size_t)n0 : (size_t)n0 * g.K) + stepB * kb0);
    const unsigned lds_base = (unsigned)(uintptr_t)LDS_PTR(char, smem);
    // one tile alone reads these weights: streaming loads, which push nothing out of the caches (forward: see stream_weights)
    const bool once = mte == 1 && (C::B_TRANS ? g.stream_weights != 0 : streaming);
    auto issue = [&](int li) {                          // block li of this range into ring slot li % STAGES
        if (li == nk - 1 && rem < BK) {
            clamp_offsets<false, BM, 4, C::LA, BK>(rem, g.K, wave, lane, va);
            clamp_offsets<C::B_TRANS, C::BN, 4, C::LB, BK>(rem, ldb, wave, lane, vb);
        }
        const unsigned dst = lds_base + (li % STAGES) * C::STAGE_BYTES + wave * 1024;
        const u16 *sa = qa, *sb = qb;
#pragma unroll
        for (int i = 0; i < C::LA; ++i) {
            const unsigned off = va[i];
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(dst + i * 4096), "v"(off), "s"(sa) : "memory");
        }
        if (once) {
#pragma unroll
            for (int i = 0; i < C::LB; ++i) {
                const unsigned off = vb[i];
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt" :: "s"(dst + C::A_BYTES + i * 4096), "v"(off), "s"(sb) : "memory");
            }
        } else {
#pragma unroll
            for (int i = 0; i < C::LB; ++i) {
                const unsigned off = vb[i];
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(dst + C::A_BYTES + i * 4096), "v"(off), "s"(sb) : "memory");
            }
        }
        qa += BK;
        qb += stepB;
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < nk) issue(s);

    // ---- places of the operands in LDS
    const int r0 = wave / C::WN * (TM * 32), c0 = wave % C::WN * (TN * 32);    // this wavefront's first row and column of the tile
    int offA[TM], offB[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) offA[i] = (r0 + i * 32 + (lane & 31)) * (BK * 2) + ((((lane >> 5)) ^ swz<BK>(lane & 31)) << 4);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        if constexpr (!C::B_TRANS) {
            offB[j] = (c0 + j * 32 + (lane & 31)) * (BK * 2) + ((((lane >> 5)) ^ swz<BK>(lane & 31)) << 4);
        } else {
            const int s = lane & 15, col = c0 + j * 32 + ((lane >> 4) & 1) * 16 + 4 * (s & 3);
            offB[j] = ((lane >> 5) * 8 + (s >> 2)) * (C::BN * 2) + ((swap13(col >> 3) ^ (2 * (s >> 2))) << 4) + (col & 7) * 2;
        }
    }
    auto fetchB = [&](const char* t, int j, int ks) -> bf16x8 {
        if constexpr (!C::B_TRANS) return *(const bf16x8*)(t + (offB[j] ^ (ks << 5)));
        else {
            const char* p = t + offB[j] + ks * 16 * (C::BN * 2);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, p + 4 * (C::BN * 2)));
            return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    };
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    const int tm_act = min(TM, max(0, (Mt - r0 + 31) / 32));    // blocks of this wavefront that hold a row

    // ---- main loop: one barrier per block, after which its loads have landed for every wavefront and the slot of the block before
    // it is free
    for (int li = 0; li < nk; ++li) {
        wait_groups<PER, STAGES - 2>(min(nk - 1 - li, STAGES - 2));
        __builtin_amdgcn_s_waitcnt(0xc07f);             // own reads of the block before are complete (lgkmcnt only)
        __builtin_amdgcn_s_barrier();
        if (li + STAGES - 1 < nk) issue(li + STAGES - 1);
        const char* tA = smem + (li % STAGES) * C::STAGE_BYTES;
        const char* tB = tA + C::A_BYTES;
        const int steps = li == nk - 1 ? rem / 16 : KS;
        auto step = [&](int ks) {
            bf16x8 b[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = fetchB(tB, j, ks);
#pragma unroll
            for (int i = 0; i < TM; ++i)
                if (BM == 32 || i < tm_act) {
                    const bf16x8 a = *(const bf16x8*)(tA + (offA[i] ^ (ks << 5)));
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a, acc[i][j], 0, 0, 0);
                }
        };
        if (steps == KS) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) step(ks);
        } else {
            for (int ks = 0; ks < steps; ++ks) step(ks);
        }
    }

    // ---- slices: all but the last to arrive leave their sums, the last adds them up in order
    if (slices > 1) {
        const long id = (long)__builtin_amdgcn_readfirstlane(sg.first) * ntn + (long)nt * mte + mt;   // the tile's number among all
        float* const part = (float*)g.sk_part + (size_t)id * slices * (BM * C::BN);
        float* const mine = part + (size_t)slice * (BM * C::BN) + tid;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            if (i < tm_act)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        __hip_atomic_store(mine + ((i * TN + j) * 16 + v) * 256, acc[i][j][v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // arrived where the XCDs' caches meet ...
        int* const s_last = (int*)smem;
        __syncthreads();                                   // ... for every wavefront (and the ring is idle)
        if (tid == 0)
            *s_last = (__hip_atomic_fetch_add(g.sk_flags + id, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (kPartialReady - 1)) == slices - 1;
        __syncthreads();
        if (!*s_last) return;
        if (tid == 0) __hip_atomic_store(g.sk_flags + id, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // as the next launch expects
        constexpr int AT_ONCE = 4;                         // slices whose loads are in flight together
#pragma unroll
        for (int i = 0; i < TM; ++i)
            if (i < tm_act)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    f32x16 sum = {};
                    for (int s0 = 0; s0 < slices; s0 += AT_ONCE) {
                        float f[AT_ONCE][16];
#pragma unroll
                        for (int u = 0; u < AT_ONCE; ++u)
#pragma unroll
                            for (int v = 0; v < 16; ++v)
                                f[u][v] = __hip_atomic_load(part + (size_t)min(s0 + u, slices - 1) * (BM * C::BN) + tid + ((i * TN + j) * 16 + v) * 256,
                                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                        for (int u = 0; u < AT_ONCE; ++u)
                            if (s0 + u < slices) {
#pragma unroll
                                for (int v = 0; v < 16; ++v) sum[v] += f[u][v];
                            }
                    }
                    acc[i][j] = sum;
                }
    }

    // ---- results: value v of lane l is row l % 32, column (v / 4) * 8 + (l / 32) * 4 + v % 4 of the wavefront's 32 x 32 block.  Two
    // groups of four columns, 8 apart, in a wavefront's two halves become eight consecutive columns per lane; the tile is put
    // together in LDS so that memory sees whole rows of it: 256 bytes in a row (in pieces of 32 bytes, straight from the registers,
    // the stores of 67 MB took 52 us longer than none).
    const int half = lane >> 5;
    char* const out1 = smem + (r0 + (lane & 31)) * C::PITCH + (C::DGELU ? (c0 + half * 4) * 4 : (c0 + half * 8) * 2);
    auto put = [&](char* at, const unsigned (&w)[4][2]) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const auto r0 = __builtin_amdgcn_permlane32_swap(w[2 * p][0], w[2 * p + 1][0], false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(w[2 * p][1], w[2 * p + 1][1], false, false);
            *(uint4*)(at + p * 32) = make_uint4(r0[0], r1[0], r0[1], r1[1]);
        }
    };
    __syncthreads();                                        // every wavefront is done with the ring
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int cj = c0 + j * 32;
        if (cj >= Nt) break;                                // (widths are multiples of 32: all of a block's columns or none)
        float bias[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) bias[v] = 0.f;
        if constexpr (C::B_TRANS) {
            if (g.bias) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint2 w = *(const uint2*)((const u16*)g.bias + (size_t)e * g.Nout + n0 + cj + q * 8 + half * 4);
                    bias[4 * q] = __uint_as_float(w.x << 16);  bias[4 * q + 1] = __uint_as_float(w.x & 0xffff0000u);
                    bias[4 * q + 2] = __uint_as_float(w.y << 16);  bias[4 * q + 3] = __uint_as_float(w.y & 0xffff0000u);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (i >= tm_act) break;
            if constexpr (C::DGELU) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(float4*)(out1 + i * 32 * C::PITCH + j * 128 + q * 32) =
                        make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
                continue;
            }
            unsigned w[4][2], w2[4][2];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float x[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] = acc[i][j][4 * q + t] + bias[4 * q + t];
                w[q][0] = pack_bf16x2(x[0], x[1]);
                w[q][1] = pack_bf16x2(x[2], x[3]);
                if constexpr (KIND == kRowsNN_GeLU) {
                    float h[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) h[t] = x[t] * normal_cdf(x[t]);
                    w2[q][0] = pack_bf16x2(h[0], h[1]);
                    w2[q][1] = pack_bf16x2(h[2], h[3]);
                }
            }
            put(out1 + i * 32 * C::PITCH + j * 64, w);
            if constexpr (KIND == kRowsNN_GeLU) put(out1 + (BM + i * 32) * C::PITCH + j * 64, w2);
        }
    }
    __syncthreads();
    const int piece = tid & 15, prow = tid >> 4;            // 16 pieces of 16 bytes make a row of the tile; 16 rows at a time
    const bool pok = piece * 8 < Nt;
#pragma unroll
    for (int r = 0; r < BM; r += 16) {
        const int m = r + prow;
        if (m < Mt && pok) {
            size_t row = (size_t)row0 + m;
            const char* const from = smem + m * C::PITCH + piece * (C::DGELU ? 32 : 16);
            if constexpr (C::DGELU) {                       // dZ = dH (Phi(z) + z phi(z))
                const size_t o = row * g.Nout + n0 + piece * 8;
                const uint4 zw = *(const uint4*)((const u16*)g.Zin + o);
                const float4 lo = *(const float4*)from, hi = *(const float4*)(from + 16);
                const unsigned w[4] = {zw.x, zw.y, zw.z, zw.w};
                float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float zf = __uint_as_float(t & 1 ? w[t / 2] & 0xffff0000u : w[t / 2] << 16);
                    x[t] *= gelu_slope(zf);
                }
                store_out((uint4*)((u16*)g.C + o), make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])), streaming);
                continue;
            }
            if constexpr (KIND == kRowsNN_GeLU)
                store_out((uint4*)((u16*)g.C2 + row * g.Nout + n0 + piece * 8), *(const uint4*)(from + BM * C::PITCH), streaming);
            if constexpr (KIND == kRowsNN) {                // top-1: the row goes straight to its token's place in Y
                if (g.c_scatter) row = g.c_scatter[row];
            }
            store_out((uint4*)((u16*)g.C + row * g.Nout + n0 + piece * 8), *(const uint4*)from, streaming);
        }
    }
}

template <int KIND, int BM, int STAGES, int OCC>
void launch_tile_cfg(const GemmArgs& a, hipStream_t st)
{
    using C = TileCfg<KIND, BM, STAGES>;
    constexpr auto kern = ggemm_tile_kernel<KIND, BM, STAGES, OCC>;
    if (!allow_dynamic_lds<kern>(C::SMEM)) return;
    const int nk = (a.K + C::BK - 1) / C::BK;
    const long tiles = most_tiles(a, BM);
    long slices = 1;
    // As many slices as keep all workgroups on the chip at once, and no more than 640 of them: every slice leaves its sums in memory (8
    // tokens, 16 experts, d 1024, h 4096, tiles of 32: FC1 and FC2 26 and 27 us cut for 1024 workgroups, 23.5 and 24 for 640).
    if (tiles <= kSkPhases * kMaxPersistentWgs) {       // (one arrival counter per tile)
        slices = std::min<long>({std::min(256L * OCC, 640L) / tiles, 16, nk / 4});   // (far below kPartialReady arrivals)
        const long room = (long)(kSkPhases * kMaxPersistentWgs * kPartialBytesPerWg) / (tiles * BM * C::BN * 4);
        slices = std::max<long>(1, std::min(slices, room));
    }
    const long units = tiles * slices;
    hipLaunchKernelGGL(kern, dim3((unsigned)((units + 7) / 8 * 8)), dim3(C::NT), C::SMEM, st, a, (a.Nout + C::BN - 1) / C::BN, (int)slices);
}

template <int KIND> void launch_tile(const GemmArgs& a, hipStream_t st)
{
    const int BM = small_tile_height(a);
    if (BM == 32) launch_tile_cfg<KIND, 32, 2, 4>(a, st);
    else if (BM == 64) launch_tile_cfg<KIND, 64, 2, 3>(a, st);
    else launch_tile_cfg<KIND, 128, 2, 2>(a, st);
}
}  // namespace sk
}  // namespace moe
