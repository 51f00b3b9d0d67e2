// How operand tiles lie in LDS, and the fragment reads out of them, for the GEMM kernels whose waves own 128 rows x 32 NB
// columns of the output (gfx950).
//   K-contiguous operand: slabs of EXT rows x 128 bytes (a pair of stages of 64 along K);
//   MN-contiguous operand: slabs of 64 K-rows x EXT bytes (a stage).
#pragma once

#include "gemm_common.hpp"

namespace fp8mm {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

#ifndef LDS_PTR
#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))
#endif

// Chunk swizzles.  K-contiguous slab: rows of 128 B = 8 chunks; MN-contiguous slab: rows of
// EXT bytes = 16 or 8 chunks (the swizzle value is reduced to the chunk count).  Measured on gfx950: with these a 16-byte fragment read costs 5 clocks per
// wave instruction (the conflict-free rate, 64 banks of 4 bytes) and a transposing 8-byte read
// 7.3 clocks.
__device__ __forceinline__ int swz_kc(int row) { return (row >> 1) & 7; }
// MN-contiguous slab: mc_pos = position in its K-row of the chunk whose index in memory is c; mc_mem
// = the memory chunk that sits at position p (the inverse map, used on the global side of the direct
// loads, whose LDS placement is fixed).  The XOR with the K-row spreads the 8 K-rows that one 16-lane
// group of a transposing read touches over 8 chunk positions.  In a 256-byte row (16 chunks, all 64
// banks) the odd memory chunks also change halves: the two 16-lane groups that are served
// together read neighbouring chunks (columns 0-15 and 16-31 of a block), which then lie in
// different halves of the banks instead of sharing 32 of them.
template <int CH>
__device__ __forceinline__ int mc_pos(int c, int krow)
{
    const int p = c ^ (krow & 7 & (CH - 1));
    return CH == 16 ? p ^ ((c & 1) << 3) : p;
}
template <int CH>
__device__ __forceinline__ int mc_mem(int p, int krow)
{
    const int c = p ^ (krow & 7 & (CH - 1));               // right but for bit 3, which does not enter bit 0
    return CH == 16 ? c ^ ((c & 1) << 3) : c;
}

// Rows of a K-contiguous slab / bytes of a K-row of the other kind in LDS.  192 columns of the other kind lie in rows of 256
// bytes: the columns of either wave begin at a half, so that the swizzle and the address arithmetic are those of 256
// columns; the last quarter of a half repeats the chunk before it (the same lines are asked for, nothing more is read).
template <bool KC, int EXT>
constexpr int lds_extent() { return !KC && EXT == 192 ? 256 : EXT; }

// Per-lane LDS offset of the first fragment read of an operand whose slabs begin at `region`; wsel: which half of the
// rows / columns the wave takes.  EXT: rows of a K-contiguous slab, bytes of a K-row of the other kind.
template <bool KC, int EXT>
__device__ __forceinline__ unsigned fragment_start(unsigned region, int wsel, int l)
{
    const int h = l >> 5;
    if (KC) {
        // lane = (r = l % 32, h = l / 32) reads K bytes 32h .. 32h+31 of row r of its stage:
        // chunks 4 par + 2h and + 1 of the 128-byte row (par = stage parity)
        const int row = wsel * (EXT / 2) + (l & 31);
        return region + row * 128 + (((2 * h) ^ swz_kc(row)) * 16);
    }
    // lane = (r = l % 32, h): column r, K bytes 32h .. 32h+31, gathered by four transposing
    // reads of 8 K-rows x 16 columns per 16-lane group; lanes 2q and 2q+1 address K-row q
    constexpr int CH = EXT / 16;
    const int t16 = l & 15, gq = (l >> 4) & 1;
    const int krow = 32 * h + (t16 >> 1);
    return region + krow * EXT + mc_pos<CH>(wsel * (CH / 2) + gq, krow) * 16 + (t16 & 1) * 8;
}

// One read-part of the fragment reads of stage kt for one operand: 16 bytes per lane of block blk
// (half 0 or 1 of the lane's 32 bytes), as one 16-byte read (KC) or two transposing reads (MC).
// EXT: rows of a K-contiguous slab, bytes of a K-row of the other kind (lds_extent); MC_SLOTS: slabs in the ring of the other kind.
// rd: see fragment_start.
template <bool KC, int EXT, int MC_SLOTS>
__device__ __forceinline__ void read_part(const uint8_t* smem, unsigned rd, int kt, int kc_slot, int blk, int half, v8i* f)
{
    if (KC) {
        const unsigned addr = (rd ^ (unsigned)((kt & 1) * 64 + half * 16)) + kc_slot * (EXT * 128) + blk * 32 * 128;
        const v4i a = *LDS_PTR(v4i, smem + addr);
        f[blk][4 * half + 0] = a.x; f[blk][4 * half + 1] = a.y; f[blk][4 * half + 2] = a.z; f[blk][4 * half + 3] = a.w;
    } else {
        const unsigned base = (unsigned)(kt & (MC_SLOTS - 1)) * (64 * EXT) + (rd ^ (unsigned)(blk * 32));
#pragma unroll
        for (int s = 2 * half; s < 2 * half + 2; ++s) {
            const v2i p = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_PTR(v2i, smem + base + s * 8 * EXT));
            f[blk][2 * s] = p.x; f[blk][2 * s + 1] = p.y;
        }
    }
}

}  // namespace
}  // namespace fp8mm
