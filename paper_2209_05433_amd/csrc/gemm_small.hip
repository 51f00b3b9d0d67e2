// Matrix-core GEMM for small problems, any shape and any alignment, for gfx950 (MI355X).
//
//   c[M x N] = (op(A)[M x K] x op(B)[K x N]) / (sA sB),   D = cast_out(c)
//
// The tiled kernel wants hundreds of 256-wide output tiles; a batch of a few tokens, or a 256 x 256
// product, gives it a handful of workgroups that each walk all of K behind 160 KB of LDS.  Here the
// output tile is 32 x 32, 32 x 64 or 64 x 64, and the waves of a workgroup share its K: wave w takes
// the chunks w, w + NW, ... of 64 or 128, so that
//   - a few hundred workgroups exist where the tiled kernel has ten, and K is walked NW times faster;
//   - every byte is read once per workgroup, by the one wave that multiplies it: nothing is shared
//     between waves until the end, and there is no barrier in the K loop;
//   - D chunks of both operands (two; one with 64 x 64 tiles, of 64 or 128) are in flight per wave, in registers.
// A chunk is fetched as it lies in memory, neighbouring lanes on neighbouring 16 bytes of a row (loads
// at any address; pieces that reach over an edge load the last 16 bytes of their row and shift), and
// goes into a slab of LDS that belongs to the wave, out of which the fragments of the matrix
// instruction are read: 16-byte reads for an operand that is contiguous along K, transposing reads for
// the other kind.  (Loading the K-contiguous kind straight into the fragment layout, a row per lane,
// needs no LDS but touches 64 lines per instruction, which the vector cache looks up one per clock:
// 16 x 12288 x 12288 took 51 us, this form 34 us = 4.4 TB/s.)  At the end the waves' sums meet in LDS, are
// added in wave order and leave through the same steps as in the tiled kernel (arXiv 2209.05433,
// Section 2: factors taken out once per output; for the products see the ACC_* constants).
//
// Bound by latency where a form has less than a workgroup per compute unit (256 x 256 x 256: 8.6 us on
// the tiled kernel, 3.9 here), by the stream of the weight for few tokens (16 x 6144 x 2048: 25 -> 5.7 us;
// 16 x 12288 x 12288: 107 -> 34), by LDS and vector instructions per product beyond that (64 x 64 tiles
// reach 0.8 PFLOP/s; 1024 x 1024 x 1024: 17.8 -> 8.5 us; 1000 x 3000 x 1000: 53 -> 18).
//
// This file is compiled once per pair of storage orders: -DFP8MM_LAYOUT.
#include "gemm_small_tile.hpp"

#include <atomic>

namespace fp8mm {
namespace {

// Tile of 32 RM x 32 RN outputs, NW waves, D chunks in flight per wave.
template <int FMT_A, int FMT_B, int ACC, bool A_KC, bool B_KC, int RM, int RN, int S, int NW, int D>
__global__ __launch_bounds__(64 * NW) void gemm_small_kernel(
    const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, void* __restrict__ C,
    int64_t M, int64_t N, int64_t K, EpilogueArgs ep)
{
    typedef Operand<A_KC, RM, S> OpA;
    typedef Operand<B_KC, RN, S> OpB;
    constexpr int CK = S * SK;
    constexpr int PER_WAVE = small_lds_per_wave<A_KC, B_KC, RM, RN, S>();
    constexpr int RED = 32 * RM * RED_PITCH * 4;          // bytes of a wave's sums
    static_assert(PER_WAVE - RED >= 32 * (RM + RN) * 8, "the reciprocals of the factors lie behind the first wave's sums");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];       // NW * PER_WAVE
    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Tiles down the rows of C first; every XCD (workgroup ids go round-robin over the 8 of them) gets one
    // contiguous run, so that the tiles of one column strip share their B in one L2.
    const int64_t tiles_m = (M + 32 * RM - 1) / (32 * RM), total = gridDim.x;
    const int64_t x = blockIdx.x % 8, idx = blockIdx.x / 8, share = total / 8, rem = total % 8;
    const int64_t p = x * share + (x < rem ? x : rem) + idx;
    const int64_t m0 = (p % tiles_m) * (32 * RM), n0 = (p / tiles_m) * (32 * RN);

    // the factors that the thread will take the reciprocals of, loaded while the products run
    const float sA_host = ep.sA, sB_host = ep.sB;         // by value: a choice between two memory locations would cost scratch
    const bool uniform = !ep.a_per_row && !ep.b_per_col;
    constexpr int FACTORS = (RM + RN + 2 * NW - 1) / (2 * NW);            // per thread
    float factor[FACTORS];
#pragma unroll
    for (int f = 0; f < FACTORS; ++f) {
        const int t = tid + f * 64 * NW;
        factor[f] = 1.0f;
        if (ep.a_per_row && t < 32 * RM) factor[f] = ep.sA_dev[m0 + t < M ? m0 + t : M - 1];
        if (ep.b_per_col && t >= 32 * RM && t < 32 * (RM + RN)) factor[f] = ep.sB_dev[n0 + t - 32 * RM < N ? n0 + t - 32 * RM : N - 1];
    }

    OpA a; OpB b;
    a.setup(A, M, K, m0, l);
    b.setup(B, N, K, n0, l);
    uint8_t* slab_a = lds + w * PER_WAVE;
    uint8_t* slab_b = slab_a + OpA::SLAB;

    v16f acc[RN][RM];
#pragma unroll
    for (int i = 0; i < RN; ++i)
#pragma unroll
        for (int j = 0; j < RM; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    auto multiply = [&](const u32x4 (&xa)[OpA::PIECES], const u32x4 (&xb)[OpB::PIECES]) __attribute__((always_inline)) {
        a.store(xa, slab_a, l);
        b.store(xb, slab_b, l);
#pragma unroll
        for (int sub = 0; sub < S; ++sub) {
            v8i fa[RM], fb[RN];
            a.fragments(slab_a, sub, l, fa);
            b.fragments(slab_b, sub, l, fb);
            if (ACC == ACC_FP8) {
#pragma unroll
                for (int i = 0; i < RN; ++i)
#pragma unroll
                    for (int j = 0; j < RM; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[i], fa[j], acc[i][j], FMT_B, FMT_A, 0, 0, 0, 0);
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    v8h ha[RM], hb[RN];
#pragma unroll
                    for (int j = 0; j < RM; ++j) ha[j] = widen8<FMT_A>(fa[j][2 * s], fa[j][2 * s + 1]);
#pragma unroll
                    for (int i = 0; i < RN; ++i) hb[i] = widen8<FMT_B>(fb[i][2 * s], fb[i][2 * s + 1]);
#pragma unroll
                    for (int i = 0; i < RN; ++i)
#pragma unroll
                        for (int j = 0; j < RM; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hb[i], ha[j], acc[i][j], 0, 0, 0);
                }
            }
        }
    };

    // Chunks that lie inside K: no tests, and a load for every step (the last ones repeat the wave's
    // last chunk), so that the waits leave D - 1 chunks in flight.
    const int64_t chunks = (K + CK - 1) / CK;
    const int64_t plain = (A_KC || M >= 16) && (B_KC || N >= 16) ? K / CK : 0;
    const int64_t mine = plain > w ? (plain - w + NW - 1) / NW : 0;      // of this wave
    if (mine > 0) {
        u32x4 xa[D][OpA::PIECES], xb[D][OpB::PIECES];
        auto fetch = [&](int d, int64_t i) __attribute__((always_inline)) {
            const int64_t c = w + NW * (i < mine ? i : mine - 1);
            a.fetch(xa[d], c);
            b.fetch(xb[d], c);
        };
#pragma unroll
        for (int d = 0; d < D; ++d) fetch(d, d);
        int64_t i = 0;
        for (; i + D <= mine; i += D)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                multiply(xa[d], xb[d]);
                fetch(d, i + d + D);
            }
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (i + d < mine) multiply(xa[d], xb[d]);
    }
    for (int64_t c = plain + (w + NW - plain % NW) % NW; c < chunks; c += NW) {
        u32x4 xa[OpA::PIECES], xb[OpB::PIECES];
        a.fetch_guarded(xa, c, l);
        b.fetch_guarded(xb, c, l);
        multiply(xa, xb);
    }

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
        if (i == 0 && !uniform) {
#pragma unroll
            for (int f = 0; f < FACTORS; ++f)
                if (tid + f * 64 * NW < 32 * (RM + RN)) *LDS_PTR(double, row_factors + tid + f * 64 * NW) = 1.0 / factor[f];
        }
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
        unsigned* cells = (unsigned*)(lds + (NW > 1 ? PER_WAVE + RED : 0));   // behind the second wave's sums; a lone wave's have been read
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

template <int FA, int FB, int ACC, bool A_KC, bool B_KC, int RM, int RN, int S, int NW, int D>
int launch_form(const GemmArgs& g)
{
    constexpr int LDS = NW * small_lds_per_wave<A_KC, B_KC, RM, RN, S>();
    auto kern = gemm_small_kernel<FA, FB, ACC, A_KC, B_KC, RM, RN, S, NW, D>;
    if (LDS > 65536) {
        // more dynamic LDS than the default limit: raised once per device
        static std::atomic<unsigned long long> attr_set{0ull};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return fail(FP8_ERR_DEVICE, "hipGetDevice failed");
        const unsigned long long bit = 1ull << (dev & 63);
        if (dev >= 64 || !(attr_set.load(std::memory_order_relaxed) & bit)) {
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
            if (e != hipSuccess) return fail(FP8_ERR_DEVICE, "hipFuncSetAttribute(LDS=%d): %s", LDS, hipGetErrorString(e));
            if (dev < 64) attr_set.fetch_or(bit, std::memory_order_relaxed);
        }
    }
    const int64_t tiles = ((g.M + 32 * RM - 1) / (32 * RM)) * ((g.N + 32 * RN - 1) / (32 * RN));
    enqueue(kern, dim3((unsigned)tiles), dim3(64 * NW), LDS, g.stream, g.A, g.B, g.C, g.M, g.N, g.K, g.ep);
    return check_launch("gemm (small tiles)");
}

template <int FA, int FB, int ACC>
int launch_acc(const GemmArgs& g, int form)
{
    constexpr bool A_KC = (FP8MM_LAYOUT & 2) == 0, B_KC = (FP8MM_LAYOUT & 1) != 0;
    // (waves, chunks of 64 or 128 and chunks in flight measured best of about twenty combinations)
    switch (form) {
        case SMALL_32x32: return launch_form<FA, FB, ACC, A_KC, B_KC, 1, 1, 2, 8, 2>(g);
        case SMALL_32x64: return launch_form<FA, FB, ACC, A_KC, B_KC, 1, 2, 2, 4, 2>(g);
    }
    // Both operands contiguous along K: chunks of 128 read whole lines and take half the trips.  Eight waves where a compute unit
    // has one tile, whose four waves keep 32 KB in flight, a quarter of what the stream of a weight takes (64 x 12288 x 12288
    // 63 -> 43 us, FP8 mode 50 -> 42; 256 x 3072 x 12288 56 -> 32, 41 -> 30; 512 x 2048 x 6144 27 -> 20; 64 x 12288 x 3072
    // 21 -> 15); four where it has several and K is long (128 x 12288 x 12288 84 -> 63, FP8 mode 76 -> 61; 512 x 3072 x 12288
    // 72 -> 57).  The first form stays where K is short (512 x 6144 x 2048: 21.7, here 22.7: three workgroups a compute
    // unit against two; the dispatcher's table tells them apart) and for the other orders, whose slabs of 128 x 64 leave room for one workgroup.
    if constexpr (A_KC && B_KC) {
        if (form == SMALL_64x64_LINES8) return launch_form<FA, FB, ACC, A_KC, B_KC, 2, 2, 2, 8, 1>(g);
        if (form == SMALL_64x64_LINES4) return launch_form<FA, FB, ACC, A_KC, B_KC, 2, 2, 2, 4, 1>(g);
    }
    // K of one chunk, or two, and more tiles than run at once (four a compute unit): as many waves.  The others would have nothing to multiply, and their zeros
    // would be added; the sums are the same bit for bit.  5 x 300000 x 64 stored K x M 34 -> 14 us, 1500000 x 10 x 100 186 -> 110; with fewer tiles the
    // end of a tile is what takes long, and goes faster with four waves (2064 x 400 x 64: 5.4 us, 6.9 with one).
    if (((g.M + 63) / 64) * ((g.N + 63) / 64) > 4 * 256) {
        if (g.K <= SK) return launch_form<FA, FB, ACC, A_KC, B_KC, 2, 2, 1, 1, 1>(g);
        if (g.K <= 2 * SK) return launch_form<FA, FB, ACC, A_KC, B_KC, 2, 2, 1, 2, 1>(g);
    }
    return launch_form<FA, FB, ACC, A_KC, B_KC, 2, 2, 1, 4, 1>(g);
}

}  // namespace

#if !defined(FP8MM_LAYOUT)
#error "compile with -DFP8MM_LAYOUT=0..3 (2 * transA + transB)"
#endif

template <int FA, int FB>
static int launch_formats(const GemmArgs& g, int form)
{
    return g.acc == ACC_FP8 ? launch_acc<FA, FB, ACC_FP8>(g, form) : launch_acc<FA, FB, ACC_F16>(g, form);
}

int FP8MM_SMALL_NAME(FP8MM_LAYOUT)(const GemmArgs& g, int form)
{
    if (g.fmtA == FP8_E4M3)
        return g.fmtB == FP8_E4M3 ? launch_formats<FP8_E4M3, FP8_E4M3>(g, form) : launch_formats<FP8_E4M3, FP8_E5M2>(g, form);
    return g.fmtB == FP8_E4M3 ? launch_formats<FP8_E5M2, FP8_E4M3>(g, form) : launch_formats<FP8_E5M2, FP8_E5M2>(g, form);
}

}  // namespace fp8mm
