// The epilogue of the GEMM kernels whose workgroups of four waves own 256 rows x 64 NB columns of C, each
// wave 128 x 32 NB of them as NB x 4 blocks of 32 x 32 (gfx950).
#pragma once

#include "gemm_common.hpp"

#include <type_traits>

namespace fp8mm {
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

// LDS of the epilogue: the waves' blocks (at most 4 x 32 rows of 528 bytes), then these.
constexpr int EP_COLUMNS = 72 * 1024;       // reciprocals of the per-column factors, 256 floats or doubles
constexpr int EP_AMAX = 74 * 1024;          // one word per wave

// The accumulators of one wave -> memory.
//   c = acc * ra(row) [* cb(column)]: the reciprocal scales, applied once per output.  With per-column
//   factors F64 keeps both reciprocals and their product in 64 bits, rounded once: as accurate as dividing by
//   the product, and finite wherever that is (1 / sA alone may lie beyond the 32-bit range);
//   amax of |c| (if asked for); conversion to the output kind; whole-line stores.
// A lane holds 4 consecutive N of one C row per accumulator quad; written straight out that would
// be small pieces scattered over 32 rows per instruction.  Instead the wave turns each 32 x 32 NB
// block around through its own piece of the (now idle) LDS and stores it with 16 bytes per lane
// along N: whole 128-byte lines where the rows of C start on them (64-byte halves for FP8 outputs of the
// narrow tile).  Rows that start anywhere take the same stores: at any address they are one instruction
// (element by element, 4096 x 50257 x 2048 with bf16 output took 889 us against 711 us for N = 50272).
// Every output kind is converted before the turn (FP8: multiplied by the output scale and rounded sixteen at
// a time by the routine of the cast kernels), so the turn moves 4, 2 or 1 bytes per output.
// All four waves call it (barriers inside where there are per-column factors or an output maximum).
template <int OUT, bool BVEC, int NB, bool F64>
__device__ __forceinline__ void epilogue(v16f (&acc)[NB][4], uint8_t* smem, const EpilogueArgs& ep, void* C, int M, int N,
                                         int m0, int n0, int w, int l)
{
    constexpr bool FP8OUT = OUT == OUT_E4M3 || OUT == OUT_E5M2;
    constexpr int FMT = OUT == OUT_E5M2 ? FP8_E5M2 : FP8_E4M3;
    constexpr int ESZ = OUT == OUT_F32 ? 4 : OUT == OUT_BF16 ? 2 : 1;     // bytes per output
    constexpr int WN = 32 * NB;                                           // columns of the wave's sub-tile
    constexpr int ROWB = WN * ESZ + 16;                                   // padded LDS row of the wave's block
    constexpr int LANES = WN * ESZ / 16;                                  // lanes that hold a row of it between them
    constexpr int ROWS_PER_ST = 64 / LANES;                               // C rows covered by one store instruction
    const int h = l >> 5, wn = w & 1;
    const int wave_m0 = m0 + (w >> 1) * 128, wave_n0 = n0 + wn * WN;

    // reciprocal scales: per row in ra (with the per-tensor sB folded in), per column in LDS, one division
    // per column of the tile (64 per lane, kept in registers, were a microsecond of the tile's end)
    // (the by-value factors are copied out of the argument block first: a choice between two
    // memory locations would force the block into scratch memory)
    const float sA_host = ep.sA, sB_host = ep.sB;
    float ra[4];
    double ra64[4];
    {
        const double b = BVEC ? 1.0 : (double)scale_value(ep.sB_dev, sB_host);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
            const float a = ep.a_per_row ? ep.sA_dev[min(wave_m0 + mb * 32 + (l & 31), M - 1)] : scale_value(ep.sA_dev, sA_host);
            ra64[mb] = 1.0 / ((double)a * b);
            ra[mb] = (float)ra64[mb];
        }
    }
    typedef typename std::conditional<F64, double, float>::type factor_t;
    typedef factor_t v4factor __attribute__((ext_vector_type(4)));
    factor_t* columns = (factor_t*)(smem + EP_COLUMNS);
    if (BVEC) {
        const int t = w * 64 + l;
        if (t < 64 * NB) *LDS_PTR(factor_t, columns + t) = (factor_t)1 / (factor_t)ep.sB_dev[min(n0 + t, N - 1)];
        __syncthreads();
    }
    auto column_factors = [&](int nb, int q) { return *LDS_PTR(v4factor, columns + wn * WN + nb * 32 + 8 * q + 4 * h); };
    const float sD = FP8OUT ? scale_value(ep.sD_dev, 1.0f) : 1.0f;

    // Output maximum: outputs beyond the edges of C hold products of redirected loads and do not count.
    const bool n_edge = n0 + 64 * NB > N;
    unsigned amax_bits = 0;

    uint8_t* blk = smem + w * (32 * ROWB);
    uint8_t* c_wave = (uint8_t*)C + ((size_t)wave_m0 * N + wave_n0) * ESZ;
    const int st_row = l / LANES, st_col = (l % LANES) * 16;                             // byte column in memory
    const int left = l < ROWS_PER_ST * LANES ? N - (wave_n0 + st_col / ESZ) : 0;         // columns from the lane's first one to the edge
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
        unsigned row_max = 0;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float y[16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v4factor f = {1, 1, 1, 1};
                if (BVEC) f = column_factors(nb, q);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a = acc[nb][mb][4 * q + i];
                    if (!BVEC) y[4 * q + i] = a * ra[mb];
                    else if (F64) y[4 * q + i] = a * (float)(ra64[mb] * f[i]);
                    else y[4 * q + i] = a * ra[mb] * (float)f[i];
                }
            }
            unsigned quad_max = 0;                       // over the 16 outputs (FP8 outputs: also tells how to convert)
            if (FP8OUT) {
#pragma unroll
                for (int i = 0; i < 16; ++i) quad_max = max(quad_max, as_u32(y[i]) & 0x7fffffffu);
            }
            if (ep.amax_out) {
                if (n_edge) {
                    const int inside = N - (wave_n0 + nb * 32 + 4 * h);
#pragma unroll
                    for (int i = 0; i < 16; ++i) row_max = max(row_max, 8 * (i >> 2) + (i & 3) < inside ? as_u32(y[i]) & 0x7fffffffu : 0u);
                } else if (FP8OUT) {
                    row_max = max(row_max, quad_max);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) row_max = max(row_max, as_u32(y[i]) & 0x7fffffffu);
                }
            }
            uint8_t* dst = blk + (l & 31) * ROWB + (nb * 32 + 4 * h) * ESZ;
            if (OUT == OUT_F32) {
#pragma unroll
                for (int q = 0; q < 4; ++q) *LDS_PTR(v4f, dst + 8 * q * ESZ) = (v4f){y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]};
            } else if (OUT == OUT_BF16) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v2i o;
                    o.x = (int)__builtin_bit_cast(unsigned, __builtin_convertvector((v2f){y[4 * q], y[4 * q + 1]}, v2bf));
                    o.y = (int)__builtin_bit_cast(unsigned, __builtin_convertvector((v2f){y[4 * q + 2], y[4 * q + 3]}, v2bf));
                    *LDS_PTR(v2i, dst + 8 * q * ESZ) = o;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) y[i] *= sD;
                // The products are as large as the largest one, whose magnitude is known: where it is within the
                // format (a factor from the output's own maximum), nothing has to be clamped or looked at one by one.
                const float top = __builtin_fabsf(as_f32(quad_max) * sD);
                u32x4 o;
                if (top <= (FMT == FP8_E4M3 ? 448.0f : 57344.0f)) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[q] = encode4_inside<FMT>(y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]);
                } else {
                    o = encode16<FMT, kCastCvt>(y);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) *LDS_PTR(unsigned, dst + 8 * q) = o[q];
            }
        }
        if (wave_m0 + mb * 32 + (l & 31) < M) amax_bits = max(amax_bits, row_max);
#pragma unroll
        for (int i = 0; i < (32 + ROWS_PER_ST - 1) / ROWS_PER_ST; ++i) {
            const int row = i * ROWS_PER_ST + st_row;
            if (wave_m0 + mb * 32 + row >= M || left <= 0) continue;                       // beyond the edges of C
            if (32 % ROWS_PER_ST != 0 && row >= 32) continue;                              // (or of the block)
            uint8_t* out = c_wave + (size_t)(mb * 32 + row) * N * ESZ + st_col;
            const u32x4 o = *LDS_PTR(u32x4, blk + row * ROWB + st_col);
            if (left >= 16 / ESZ) {
                *(u32x4_any*)out = o;                    // (non-temporal stores measured the same, 8 shapes)
            } else {                                    // the end of a row inside the lane's 16 bytes
#pragma unroll
                for (int e = 0; e < 16 / ESZ - 1; ++e) {
                    if (e < left) {
                        if (ESZ == 4) ((unsigned*)out)[e] = o[e];
                        else if (ESZ == 2) ((unsigned short*)out)[e] = (unsigned short)(o[e >> 1] >> (16 * (e & 1)));
                        else out[e] = (uint8_t)(o[e >> 2] >> (8 * (e & 3)));
                    }
                }
            }
        }
    }
    if (ep.amax_out) {
        // one atomic per workgroup: the waves of a round end together, and a thousand atomics on one cell
        // took longer than a tile's stores
        unsigned m = amax_bits;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d, 64));
        unsigned* cells = (unsigned*)(smem + EP_AMAX);
        if (l == 0) *LDS_PTR(unsigned, cells + w) = m;
        __syncthreads();
        if (w == 0) wave_amax_commit(l < 4 ? *LDS_PTR(unsigned, cells + l) : 0u, ep.amax_out);
    }
}

// The workgroup's tile, with the output kind and the scale granularity chosen for the whole wave.  The LDS holds
// nothing any more that somebody needs.
template <int NB, bool F64>
__device__ __forceinline__ void store_tile(v16f (&acc)[NB][4], uint8_t* smem, const EpilogueArgs& ep, void* C, int M, int N, int m0, int n0, int w)
{
    // The lane index is taken afresh from the execution mask count: values derived from the one
    // computed before the K loop would have to stay in registers (or be spilled) all through it.
    const int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    if (ep.b_per_col) {
        switch (ep.out_kind) {
            case OUT_F32: epilogue<OUT_F32, true, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
            case OUT_BF16: epilogue<OUT_BF16, true, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
            case OUT_E4M3: epilogue<OUT_E4M3, true, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
            default: epilogue<OUT_E5M2, true, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
        }
    } else {
        switch (ep.out_kind) {
            case OUT_F32: epilogue<OUT_F32, false, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
            case OUT_BF16: epilogue<OUT_BF16, false, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
            case OUT_E4M3: epilogue<OUT_E4M3, false, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
            default: epilogue<OUT_E5M2, false, NB, F64>(acc, smem, ep, C, M, N, m0, n0, w, l); break;
        }
    }
}

}  // namespace
}  // namespace fp8mm
