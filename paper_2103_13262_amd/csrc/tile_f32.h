// Staging of 64 x 64 x 32 blocks of an fp32 matrix product for v_mfma_f32_32x32x2_f32 (internal; the fp32 grouped products
// and the dense gate gradients).  256 threads; an operand block of 64 rows (columns) x 32 reduction indices travels as two
// pieces of four elements per thread through registers into LDS; bf16 sources are widened on the way.
//
// LDS layouts: sources with the reduction index fastest in memory are kept as [row][36 floats], read 16 bytes per lane (4
// consecutive reduction indices: matrix step s of four takes element s of every lane); sources with the reduction index
// slowest (TRANS) as [k][72 floats], read 4 bytes per lane.  Both pitches spread a wavefront's read evenly over the banks.
#pragma once
#include "common.h"

namespace moe {
namespace tile_f32 {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int TM = 64, TN = 64, TK = 32;
constexpr int kPitchK = TK + 4;    // floats per LDS row, reduction index fastest
constexpr int kPitchR = TM + 8;    // floats per LDS row, reduction index slowest
static_assert(TM == TN, "one pitch for both operands");

template <bool TRANS> constexpr int operand_floats() { return TRANS ? TK * kPitchR : TM * kPitchK; }

__device__ __forceinline__ float4 load4(const float* p) { return *(const float4*)p; }
__device__ __forceinline__ float4 load4(const unsigned short* p)
{
    const uint2 w = *(const uint2*)p;
    return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                       __uint_as_float(w.y & 0xffff0000u));
}

// One operand's share of a thread (tid: number inside the 256).
template <bool TRANS, typename T> struct Stream {
    const T* p[2];
    int k_of[2];                     // reduction index of the piece inside a block
    long step;                       // elements from one block to the next
    // valid: rows (columns) of the tile that exist; others repeat an existing one and are never stored
    __device__ __forceinline__ void init(const T* base, long ld, int valid, int tid, const int32_t* gather, long row0, int div)
    {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if constexpr (!TRANS) {
                const int row = min((tid >> 3) + 32 * i, valid - 1);
                const long src = gather ? (long)(gather[row0 + row] / div) : (long)row;
                k_of[i] = (tid & 7) * 4;
                p[i] = base + src * ld + k_of[i];
            } else {
                const int k = (tid >> 4) + 16 * i, c = (tid & 15) * 4;
                p[i] = base + (long)k * ld + (c < valid ? c : 0);
                k_of[i] = k;
            }
        }
        step = TRANS ? (long)TK * ld : TK;
    }
    // block b; k_left: reduction indices from the block's first on that exist (<= 0: the block does not).  Pieces exist as
    // a whole or not at all: !TRANS needs reduction lengths (and row strides) that are multiples of 4.
    __device__ __forceinline__ void fetch(float4 (&r)[2], long b, int k_left) const
    {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            r[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k_of[i] < k_left) r[i] = load4(p[i] + b * step);
        }
    }
};
template <bool TRANS> __device__ __forceinline__ void stash_block(float* lds, const float4 (&r)[2], int tid)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if constexpr (!TRANS) *(float4*)(lds + ((tid >> 3) + 32 * i) * kPitchK + (tid & 7) * 4) = r[i];
        else *(float4*)(lds + ((tid >> 4) + 16 * i) * kPitchR + (tid & 15) * 4) = r[i];
    }
}
// reduction indices 8 kk + 4 (lane / 32) .. + 3 of row / column rb + lane % 32
template <bool TRANS> __device__ __forceinline__ void operand(const float* lds, int rb, int kk, int lane, float (&v)[4])
{
    if constexpr (!TRANS) {
        const float4 q = *(const float4*)(lds + (rb + (lane & 31)) * kPitchK + kk * 8 + (lane >> 5) * 4);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
        const float* q = lds + (kk * 8 + (lane >> 5) * 4) * kPitchR + rb + (lane & 31);
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = q[s * kPitchR];
    }
}

}  // namespace tile_f32
}  // namespace moe
