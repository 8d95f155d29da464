// What the bf16 products' kernels share: operand types, the places of 16-byte chunks in LDS and in memory, waits, stores (internal).
#pragma once
#include "common.h"

namespace moe {
namespace sk {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef unsigned short u16;
#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

// Results can leave the chip as streaming (non-temporal) stores: none of them is read again by the launch that writes
// it, and written the ordinary way they displace operand panels from the caches.  Measured on one machine, A against
// B: -2 % per step on the paper's shape (134 MB of weights per product), -6 % with 64 or 256 experts, the weight
// gradients' stores mattering most; but +1.5 to +3 % with 1, 2 or 4 experts of that width (8 to 32 MB), whose weights
// stay in the 32 MB of L2 whatever the stores do, so that what counts is how fast the stores are taken.  The host
// decides per launch (GemmArgs::stream_out): streaming when one product's weights exceed 48 MB.
// Weight gradients in fp32, or added to what is there, always leave as streaming stores.  A training step with streaming / ordinary stores
// below that line, us: fp32 654 / 661 (1 expert, 8192 rows, d 1024, h 4096), 535 / 539 (2 experts, 4096 rows each), 587 / 597 (4), 198 / 205 (8
// experts, d 768, h 3072), 176 / 190 (10, d 1024, h 2048), 183 / 193 (64, d 256, h 1024); added to, in fp32 or bf16: the same to 1 %.
typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
__device__ __forceinline__ void store_out(uint4* p, const uint4 v, bool streaming)
{
    if (streaming) {
        const u32x4_t w = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(w, (u32x4_t*)p);
    } else *p = v;
}
__device__ __forceinline__ int swap13(int c) { return (c & ~10) | ((c & 2) << 2) | ((c & 8) >> 2); }

template <int BK> __device__ __forceinline__ int swz(int r)
{
    if constexpr (BK == 32) return ((r >> 1) & 3) ^ ((r >> 3) & 1);
    else if constexpr (BK == 64) return (r >> 1) & 7;
    else return r & 15;   // 256-byte rows: every row starts at bank 0, 16 rows take 16 different chunk positions
}

// s_waitcnt vmcnt(N) only (export and LDS counters left at their maxima), gfx9 encoding.
template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
template <int PER, int MAXG> __device__ __forceinline__ void wait_groups(int groups)
{   // allow `groups` (0..MAXG) load groups of PER instructions each to stay in flight
    if constexpr (MAXG == 0) { wait_vmcnt<0>(); }
    else {
        if (groups >= MAXG) wait_vmcnt<PER * MAXG>();
        else wait_groups<PER, MAXG - 1>(groups);
    }
}

// Where lane `lane` of load i of one operand finds its 16-byte chunk of a reduction block: the byte offset from the operand's
// base, which moves on by a constant from block to block, so that a load needs one 32-bit register and no vector arithmetic
// (WIDE: 64 bits, for operands of 4 GB and more or rows that far apart).
//   !TRANS: src[row][k]; one load covers 64 / (BK/8) rows.
//    TRANS: src[k][row]; CPR = R/8 chunks per k-row; lane p of load j covers k-row j*(64/CPR) + p/CPR.
//   gather (!TRANS only): row r of the tile is the source's row gather[row0 + r] / div instead of row r.
template <bool TRANS, int R, int NW, int BK> struct Chunk {
    static __device__ __forceinline__ int krow(int i, int wave, int lane) { return (wave + i * NW) * (64 / (R / 8)) + lane / (R / 8); }   // TRANS
    static __device__ __forceinline__ int row(int i, int wave, int lane) { return (wave + i * NW) * (64 / (BK / 8)) + lane / (BK / 8); }  // !TRANS
    static __device__ __forceinline__ int col(int i, int wave, int lane) { return (lane % (BK / 8)) ^ swz<BK>(row(i, wave, lane)); }      // !TRANS
};
template <bool TRANS, int R, int NW, int L, int BK, typename Off>
__device__ __forceinline__ void setup_offsets(long ld, int valid, int wave, int lane, Off (&off)[L],
                                              const int32_t* gather = nullptr, long row0 = 0, int div = 1)
{
    using Ch = Chunk<TRANS, R, NW, BK>;
#pragma unroll
    for (int i = 0; i < L; ++i) {
        if constexpr (!TRANS) {
            int row = Ch::row(i, wave, lane);
            row = row < valid ? row : valid - 1;
            const Off src_row = gather ? (Off)(gather[row0 + row] / div) : (Off)row;
            off[i] = src_row * (Off)(ld * 2) + (Off)(Ch::col(i, wave, lane) * 16);
        } else {
            constexpr int CPR = R / 8;
            static_assert(CPR >= 16 && 64 % CPR == 0, "the position code needs 16 chunks per k-row");
            const int kr = Ch::krow(i, wave, lane);
            int c = swap13((lane % CPR) ^ (2 * (kr & 3)));
            c = c * 8 < valid ? c : 0;
            off[i] = (Off)kr * (Off)(ld * 2) + (Off)(c * 16);
        }
    }
}
// The last reduction block holds only `rem` of its BK indices: chunks past them are fetched from a place inside it instead
// (the matrix steps past `rem` are not computed; a step that holds it in its middle clears its operands there).
template <bool TRANS, int R, int NW, int L, int BK, typename Off>
__device__ __forceinline__ void clamp_offsets(int rem, long ld, int wave, int lane, Off (&off)[L])
{
    using Ch = Chunk<TRANS, R, NW, BK>;
#pragma unroll
    for (int i = 0; i < L; ++i) {
        if constexpr (!TRANS) {
            const int c = Ch::col(i, wave, lane);
            if (c * 8 >= rem) off[i] -= (Off)(c * 16);
        } else {
            const int kr = Ch::krow(i, wave, lane);
            if (kr >= rem) off[i] -= (Off)(kr - (rem - 1)) * (Off)(ld * 2);
        }
    }
}

// A value that is the same in all lanes, in scalar registers (what it is worked out from may have come through vector loads).
__device__ __forceinline__ unsigned long scalar(unsigned long v)
{
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return ((unsigned long)hi << 32) | lo;
}
__device__ __forceinline__ const u16* scalar(const u16* p) { return (const u16*)scalar((unsigned long)p); }

}  // namespace sk
}  // namespace moe
