// Pieces of the kernels with small output tiles, whose waves share K (gemm_small.hip, scaled_gemm_small.hip): how a chunk of an operand lies in
// LDS, and its fragments (gfx950).
#pragma once

#include "gemm_common.hpp"

namespace fp8mm {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

constexpr int SK = 64;                                    // K per sub-chunk; a chunk has S of them

// One operand of the tile: R blocks of 32 rows of op(A) / columns of op(B) from t0 on, `ext` of them in
// all; chunks of CK = 64 S along K.  KC: element (r, k) at base[r K + k]; else at base[k ext + r].
template <bool KC, int R, int S>
struct Operand {
    static constexpr int CK = S * SK;
    static constexpr int PIECES = 2 * R * S;              // 16-byte loads per lane and chunk
    static constexpr int ROWB = KC ? CK : 32 * R;         // bytes of a row of the chunk as it lies in memory
    static constexpr int ROWS = KC ? 32 * R : CK;
    static constexpr int PITCH = ROWB + 16;               // ... and in LDS (16 bytes spread the rows over the banks)
    static constexpr int SLAB = ROWS * PITCH;
    static constexpr int LPR = ROWB / 16;                 // lanes per row of a load
    static constexpr int RPL = 64 / LPR;                  // rows per load
    const uint8_t* base;                                  // KC: of the lane's first piece; MC: of its column
    int64_t ext, K;
    int last;                                             // KC: rows of the operand under the lane's first one
    int shift;                                            // MC: how far the lane's column lies in front of where its columns begin
    bool edge;                                            // MC: the tile reaches over the edge (same for all lanes)

    __device__ __forceinline__ void setup(const uint8_t* p, int64_t ext_, int64_t K_, int64_t t0, int l)
    {
        ext = ext_; K = K_;
        const int row = l / LPR, at = 16 * (l % LPR);
        if (KC) {
            const int64_t r = t0 + row < ext ? t0 + row : ext - 1;
            base = p + r * K + at;
            last = ext - 1 - r < 32 * R ? (int)(ext - 1 - r) : 32 * R;
            shift = 0; edge = false;
        } else {
            edge = t0 + 32 * R > ext;
            const int64_t own = t0 + at, col = own + 16 <= ext ? own : ext - 16;
            base = p + col;
            shift = own - col < 15 ? (int)(own - col) : 15;      // a lane wholly outside: any bytes do
            last = row;
        }
    }
    // chunk c, which lies wholly inside K
    __device__ __forceinline__ void fetch(u32x4 (&x)[PIECES], int64_t c) const
    {
#pragma unroll
        for (int q = 0; q < PIECES; ++q) {
            if (KC) x[q] = *(const u32x4_any*)(base + c * CK + (int64_t)(q * RPL < last ? q * RPL : last) * K);
            else x[q] = *(const u32x4_any*)(base + (c * CK + q * RPL + last) * ext);
        }
    }
    __device__ __forceinline__ void fetch_guarded(u32x4 (&x)[PIECES], int64_t c, int l) const
    {
#pragma unroll
        for (int q = 0; q < PIECES; ++q) {
            if (KC) {
                const int at = 16 * (l % LPR);
                x[q] = load_guarded(base - at + (int64_t)(q * RPL < last ? q * RPL : last) * K, c * CK + at, K);
            } else {
                const int64_t k = c * CK + q * RPL + last;
                // (rows of fewer than 16 bytes: the 16 up to the row's end begin in the rows before it and are shifted out like any others, unless
                // they would begin before the operand; byte by byte, 5 x 300000 x 64 stored K x M took 43 us)
                x[q] = k >= K ? (u32x4){0u, 0u, 0u, 0u}
                              : ext >= 16 || (k + 1) * ext >= 16 ? *(const u32x4_any*)(base + k * ext) : load_short(base + (16 - ext) + k * ext, (int)ext);
            }
        }
    }
    // the chunk into the wave's slab, as it lies in memory
    __device__ __forceinline__ void store(const u32x4 (&x)[PIECES], uint8_t* slab, int l) const
    {
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
            *LDS_PTR(u32x4, slab + (q * RPL + l / LPR) * PITCH + 16 * (l % LPR)) = !KC && edge ? drop_bytes(x[q], shift) : x[q];
    }
    // the fragments of sub-chunk s: lane (r, h) = (l % 32, l / 32) gets the K bytes 32 (S h + s) .. + 31 of
    // row r of each block
    __device__ __forceinline__ void fragments(const uint8_t* slab, int s, int l, v8i (&f)[R]) const
    {
        const int t16 = l & 15;
        const uint8_t* p = KC ? slab + (l & 31) * PITCH + 32 * (S * (l >> 5) + s)
                              : slab + (32 * (S * (l >> 5) + s) + (t16 >> 1)) * PITCH + 16 * ((l >> 4) & 1) + 8 * (t16 & 1);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (KC) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const u32x4 v = *LDS_PTR(u32x4, p + 32 * i * PITCH + 16 * j);
#pragma unroll
                    for (int d = 0; d < 4; ++d) f[i][4 * j + d] = (int)v[d];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const v2i t = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_PTR(v2i, p + 32 * i + 8 * j * PITCH));
                    f[i][2 * j] = t.x; f[i][2 * j + 1] = t.y;
                }
            }
        }
    }
};

constexpr int RED_PITCH = 36;                             // floats per row of a wave's 32 RM x 32 block of sums

template <bool A_KC, bool B_KC, int RM, int RN, int S>
constexpr int small_lds_per_wave()
{
    const int red = 32 * RM * RED_PITCH * 4, slabs = Operand<A_KC, RM, S>::SLAB + Operand<B_KC, RN, S>::SLAB;
    return red > slabs ? red : slabs;
}

}  // namespace
}  // namespace fp8mm
