// Pieces of the kernels with small output tiles, whose waves share K (gemm_small.hip, scaled_gemm_small.hip): how a chunk of an operand lies in
// LDS, its fragments, and the tile's end (gfx950).
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
                x[q] = k >= K ? (u32x4){0u, 0u, 0u, 0u} : ext >= 16 ? *(const u32x4_any*)(base + k * ext) : load_short(base + (16 - ext) + k * ext, (int)ext);
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

// The end of a tile of 32 RM x 32 RN outputs at (m0, n0) whose sums lie in the NW waves' accumulators; PER_WAVE bytes of LDS are each wave's.
// sA_host, sB_host: the operands' factors where ep names no place for them; factor: the row's or column's that the thread will take the reciprocal of.
template <int RM, int RN, int NW, int PER_WAVE>
__device__ __forceinline__ void small_tile_end(const v16f (&acc)[RN][RM], uint8_t* lds, void* __restrict__ C, int64_t M, int64_t N, int64_t m0, int64_t n0,
                                               const EpilogueArgs& ep, float sA_host, float sB_host, bool uniform, float factor, int tid, int l, int w)
{
    constexpr int RED = 32 * RM * RED_PITCH * 4;          // bytes of a wave's sums
    // The waves' sums meet in LDS, 32 columns at a time; a thread adds 4 consecutive columns of a row.  With factors
    // per row or column, their reciprocals (of the tile's rows, then of its columns; 1 for a factor that the
    // whole tensor has) lie behind the first wave's sums, in 64 bits: the product, rounded once, is as accurate as
    // dividing by the product of the factors, and finite wherever that is (1 / sA alone may leave the 32-bit range).
    const double a_all = ep.a_per_row ? 1.0 : (double)scale_value(ep.sA_dev, sA_host), b_all = ep.b_per_col ? 1.0 : (double)scale_value(ep.sB_dev, sB_host);
    const double r_all = 1.0 / (a_all * b_all);
    const float sD = ep.out_kind >= OUT_E4M3 ? scale_value(ep.sD_dev, 1.0f) : 1.0f;
    double* row_factors = (double*)(lds + RED);
    double* col_factors = row_factors + 32 * RM;
    const int esz = ep.out_kind == OUT_F32 ? 4 : ep.out_kind == OUT_BF16 ? 2 : 1;
    unsigned amax_bits = 0;
#pragma unroll
    for (int i = 0; i < RN; ++i) {
        __syncthreads();                                  // the slabs, or the block before, are done with
        if (i == 0 && !uniform && tid < 32 * (RM + RN)) *LDS_PTR(double, row_factors + tid) = 1.0 / factor;
        float* mine_red = (float*)(lds + w * PER_WAVE);
#pragma unroll
        for (int j = 0; j < RM; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *LDS_PTR(v4f, mine_red + (32 * j + (l & 31)) * RED_PITCH + 8 * q + 4 * (l >> 5)) =
                    (v4f){acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        __syncthreads();
        for (int u = tid; u < 32 * RM * 8; u += 64 * NW) {
            const int64_t gm = m0 + (u >> 3), gn = n0 + 32 * i + 4 * (u & 7);
            if (gm >= M || gn >= N) continue;
            const float* red = (const float*)lds + (u >> 3) * RED_PITCH + 4 * (u & 7);
            v4f s = *LDS_PTR(v4f, red);
#pragma unroll
            for (int v = 1; v < NW; ++v) s += *LDS_PTR(v4f, red + v * (PER_WAVE / 4));
            const int left = N - gn < 4 ? (int)(N - gn) : 4;
            float c[4], factors[4] = {(float)r_all, (float)r_all, (float)r_all, (float)r_all};
            if (!uniform) {
                const double ra = r_all * *LDS_PTR(double, row_factors + (u >> 3));
#pragma unroll
                for (int e = 0; e < 4; ++e) factors[e] = (float)(ra * *LDS_PTR(double, col_factors + 32 * i + 4 * (u & 7) + e));
            }
            unsigned quad_max = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                c[e] = s[e] * factors[e];
                if (e < left) quad_max = max(quad_max, as_u32(c[e]) & 0x7fffffffu);
            }
            amax_bits = max(amax_bits, quad_max);
            uint8_t* out = (uint8_t*)C + (size_t)(gm * N + gn) * esz;
            const bool vec = left == 4 && ((uintptr_t)out & (4 * esz - 1)) == 0;
            if (ep.out_kind == OUT_F32) {
                if (vec) *(v4f*)out = (v4f){c[0], c[1], c[2], c[3]};
                else for (int e = 0; e < left; ++e) ((float*)out)[e] = e == 0 ? c[0] : e == 1 ? c[1] : e == 2 ? c[2] : c[3];
            } else if (ep.out_kind == OUT_BF16) {
                const unsigned lo = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){c[0], c[1]}, v2bf));
                const unsigned hi = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){c[2], c[3]}, v2bf));
                if (vec) *(v2i*)out = (v2i){(int)lo, (int)hi};
                else for (int e = 0; e < left; ++e) ((unsigned short*)out)[e] = (unsigned short)((e < 2 ? lo : hi) >> (16 * (e & 1)));
            } else {
                // (the largest product tells whether anything has to be clamped or looked at one by one)
                const bool e4m3 = ep.out_kind == OUT_E4M3, inside = __builtin_fabsf(as_f32(quad_max) * sD) <= (e4m3 ? 448.0f : 57344.0f);
                const float y0 = c[0] * sD, y1 = c[1] * sD, y2 = c[2] * sD, y3 = c[3] * sD;
                const unsigned o = inside ? (e4m3 ? encode4_inside<FP8_E4M3>(y0, y1, y2, y3) : encode4_inside<FP8_E5M2>(y0, y1, y2, y3))
                                          : (e4m3 ? encode4<FP8_E4M3>(y0, y1, y2, y3) : encode4<FP8_E5M2>(y0, y1, y2, y3));
                if (vec) *(unsigned*)out = o;
                else for (int e = 0; e < left; ++e) out[e] = (uint8_t)(o >> (8 * e));
            }
        }
    }
    if (ep.amax_out) {
        // One atomic per workgroup: its waves end together, and so do hundreds of workgroups (one per wave took
        // longer than the product: 256 x 1024 x 4096 20.8 us against 7.1 without the maximum).
        unsigned* cells = (unsigned*)(lds + PER_WAVE + RED);            // behind the second wave's sums
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) amax_bits = max(amax_bits, (unsigned)__shfl_xor((int)amax_bits, d, 64));
        if (l == 0) *LDS_PTR(unsigned, cells + w) = amax_bits;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);            // (the compiler keeps the LDS accesses on their sides)
        __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0) only: nobody waits for the outputs' stores
        __builtin_amdgcn_s_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (w == 0) {
            unsigned m = l < NW ? *LDS_PTR(unsigned, cells + l) : 0u;
#pragma unroll
            for (int d = NW / 2; d >= 1; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d, 64));
            if (l == 0 && m > __hip_atomic_load((unsigned*)ep.amax_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax((unsigned*)ep.amax_out, m);
        }
    }
}

}  // namespace
}  // namespace fp8mm
