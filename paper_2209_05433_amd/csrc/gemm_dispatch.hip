// GEMM dispatcher and the generic kernel for gfx950 (MI355X).
//
// Shapes and pointers that meet the tiled kernel's conditions (K a multiple of 16, 16-byte aligned
// operands whose rows start on 16-byte boundaries) go to one of its instances; everything else to the
// matrix-core kernel for any shape (gemm_mfma_any.hip); small problems of either kind to the kernel of small
// tiles (gemm_small.hip) where a model of the run times says it is the faster one.  The generic kernel below (plain FMAs: any
// shape, any alignment, every storage order, the same epilogue) remains as the independent
// cross-check the tests force through a knob, and for outputs with more tiles than a grid holds
// (arXiv 2209.05433, Section 2: FP8 operands, fp32 accumulation, scales taken out once per output).
#include "gemm_common.hpp"

#include <utility>

#include <algorithm>
#include <cmath>

namespace fp8mm {
namespace {

// fp32 -> bf16 bits, round to nearest even; NaN stays NaN.
__device__ __forceinline__ unsigned bf16_bits(float f)
{
    const unsigned u = as_u32(f);
    const unsigned r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    return (u & 0x7fffffffu) > 0x7f800000u ? ((u >> 16) | 0x40u) : r;
}

// ------------------------------------------------------------------------------------------
// Generic kernel: 64 x 64 tile per 256-thread workgroup, 4 x 4 outputs per thread, operands
// decoded to fp32 (exactly) on their way into LDS, fp32 FMAs (each product of two FP8 values
// is exact in fp32, so this is fp32 accumulation of exact products as well).
// ------------------------------------------------------------------------------------------
constexpr int GT = 64, GK = 16;

template <int FMT_A, int FMT_B>
__global__ __launch_bounds__(256) void gemm_generic_kernel(
    const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, void* __restrict__ C,
    int64_t M, int64_t N, int64_t K, EpilogueArgs ep, bool transA, bool transB)
{
    __shared__ float As[GK][GT + 1];
    __shared__ float Bs[GK][GT + 1];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    // tiles are numbered row by row in the x dimension of the grid (the y dimension stops at 65 535)
    const int64_t tiles_n = (N + GT - 1) / GT;
    const int64_t m0 = (int64_t)(blockIdx.x / tiles_n) * GT, n0 = (int64_t)(blockIdx.x % tiles_n) * GT;
    float acc[4][4] = {};
    for (int64_t k0 = 0; k0 < K; k0 += GK) {
        for (int e = tid; e < GT * GK; e += 256) {
            const int r = e / GK, kk = e % GK;              // A: consecutive lanes along K
            const int64_t gm = m0 + r, gk = k0 + kk;
            As[kk][r] = (gm < M && gk < K) ? decode_fp8<FMT_A>(A[transA ? gk * M + gm : gm * K + gk]) : 0.0f;
            const int kb = e / GT, c = e % GT;              // B: consecutive lanes along N
            const int64_t gn = n0 + c, gkb = k0 + kb;
            Bs[kb][c] = (gn < N && gkb < K) ? decode_fp8<FMT_B>(B[transB ? gn * K + gkb : gkb * N + gn]) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < GK; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    const float sD = (ep.out_kind >= OUT_E4M3) ? scale_value(ep.sD_dev, 1.0f) : 1.0f;
    unsigned amax_bits = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t gm = m0 + ty * 4 + i, gn = n0 + tx * 4 + j;
            if (gm < M && gn < N) {
                const double a = ep.a_per_row ? (double)ep.sA_dev[gm] : (double)scale_value(ep.sA_dev, ep.sA);
                const double b = ep.b_per_col ? (double)ep.sB_dev[gn] : (double)scale_value(ep.sB_dev, ep.sB);
                const float c = acc[i][j] * (float)(1.0 / (a * b));
                amax_bits = max(amax_bits, as_u32(c) & 0x7fffffffu);
                const int64_t o = gm * N + gn;
                switch (ep.out_kind) {
                    case OUT_F32: ((float*)C)[o] = c; break;
                    case OUT_BF16: ((unsigned short*)C)[o] = (unsigned short)bf16_bits(c); break;
                    case OUT_E4M3: ((uint8_t*)C)[o] = (uint8_t)encode_bits<FP8_E4M3>(c * sD); break;
                    default: ((uint8_t*)C)[o] = (uint8_t)encode_bits<FP8_E5M2>(c * sD); break;
                }
            }
        }
    if (ep.amax_out) wave_amax_commit(amax_bits, ep.amax_out);
}

template <int FA, int FB>
int launch_generic(const GemmArgs& g)
{
    const int64_t tiles = ((g.N + GT - 1) / GT) * ((g.M + GT - 1) / GT);
    if (tiles > 0x7fffffffll)
        return fail(FP8_ERR_UNSUPPORTED, "gemm (generic kernel): %lld tiles of 64 x 64 exceed the grid limit", (long long)tiles);
    const dim3 grid((unsigned)tiles);
    enqueue((gemm_generic_kernel<FA, FB>), grid, dim3(256), 0, g.stream, g.A, g.B, g.C, g.M, g.N, g.K,
                       g.ep, g.transA, g.transB);
    return check_launch("gemm (generic kernel)");
}

__global__ void zero_fill_kernel(unsigned char* p, size_t nbytes)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nbytes; i += stride) p[i] = 0;
}

__global__ void zero_cell_kernel(unsigned* p) { *p = 0u; }

// The knob FP8_KNOB_GEMM_KERNEL = 1 forces the generic kernel, = 2 the any-shape matrix-core kernel.
bool force_generic() { return knob(FP8_KNOB_GEMM_KERNEL) == 1; }
bool force_mfma_any() { return knob(FP8_KNOB_GEMM_KERNEL) == 2; }

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }
inline int64_t tile_count(const GemmArgs& g, int64_t edge) { return ((g.M + edge - 1) / edge) * ((g.N + edge - 1) / edge); }

}  // namespace

TileTimes tile_times(int acc, double S)
{
    return acc == ACC_FP8 ? TileTimes{0.62 * S + 8.9, 0.58 * S + 7.5, 0.46 * S + 5.2} : TileTimes{1.21 * S + 10.0, 1.03 * S + 7.6, 0.79 * S + 6.4};
}

namespace {

// Microseconds of the any-shape kernel in tiles of 256 x `width`: rounds of 256 tiles, each its ends (by output kind: fp32, bf16, FP8
// with factors per column and the maximum) and S stages.  Fitted to both widths' times on 110 random problems (256 .. 8192 x 256 .. 12288 x
// 16 .. 8192, all storage orders and output kinds), within 6 %; the width that it names takes 0.04 % longer than the better of the two in the mean, 4 % at
// most (always 256: 39 %).
double any_us(const GemmArgs& g, int width)
{
    const double rounds = std::ceil(std::ceil(g.M / 256.0) * std::ceil((double)g.N / width) / 256.0), S = 2.0 * std::ceil(g.K / 128.0);
    const int kind = g.ep.out_kind == OUT_F32 ? 0 : g.ep.out_kind == OUT_BF16 ? 1 : 2;
    constexpr double wide[3] = {11.7, 8.5, 19.8}, narrow[3] = {6.3, 4.9, 10.8};
    return width == 256 ? 2.5 + rounds * (wide[kind] + 1.54 * S) : 2.8 + rounds * (narrow[kind] + 0.98 * S);
}

// Off the tiled kernel, calls that show their sums in 32 bits (fp32 outputs, an output maximum) stay on small tiles up to the times below (of
// any-shape kernels that took longer: rounds of 256 x 256 tiles, and of 128 x 128 ones of which several shared a compute unit): the waves of
// a small tile share K, and its shorter chains of sums are nearer to the 64-bit result (1.1e-7 against 1.5e-7 over K = 12288).  The line is a
// matter of what such calls have always had, no bound on the error: no product's sums get longer chains than they did.  The rounding of a
// 16-bit or FP8 output hides the difference, and without a maximum those go by what the
// kernels take: 1718 x 3405 x 6200 147 -> 105 us, 1903 x 3712 x 1809 54 -> 39, 6435 x 2048 x 2181 129 -> 80.
double small_line_us(const GemmArgs& g)
{
    const double rounds = std::ceil(std::ceil(g.M / 256.0) * std::ceil(g.N / 256.0) / 256.0), K = (double)g.K, S = std::ceil(K / 64.0);
    const double outputs = 1e-6 * (double)g.M * (double)g.N, ragged_a = g.transA && g.M % 16 != 0, ragged_b = !g.transB && g.N % 16 != 0;
    const double wide = rounds * (14.0 + 1.65 * S) + S * (3.0 * ragged_b + 3.1 * ragged_a * rounds);
    const double narrow = 6.9 + (g.ep.b_per_col ? 10.0 : 0.0) + std::max(0.03 * K, outputs * (1.8 + 0.0026 * K)) + S * (1.2 * ragged_b + 1.4 * ragged_a);
    return std::min(wide, narrow);
}

// Microseconds of a form of the small-tile kernel (gemm_small.hip): its ends, then the longer of one workgroup's walk along
// K (alone + alone_k K) and what the workgroups of a compute unit take together (each + per_k K, and, for each that waits for
// another, `further`, `ragged` where K ends inside a chunk).  fullest: how far the compute units that have one workgroup more than the
// average decide, up to four a unit.
// (32 x 32, 32 x 64 and 64 x 64 rows and columns; chunks of 128, of 64 the first 64 x 64 form.)
struct SmallTimes { double ends, each, per_k, alone, alone_k, further, ragged, fullest; };
constexpr SmallTimes kSmallTimes[3] = {{3.4, 0.3, 0.0025, 0.0, 0.001, 0.7, 0.8, 0.0}, {4.0, 0.6, 0.0018, 0.6, 0.0018, 0.0, 0.3, 0.0},
                                       {4.0, 1.2, 0.0026, 1.2, 0.0026, 0.0, 0.3, 0.0}};
constexpr double kPerK32Lines = 0.0014;      // per_k of the first, both operands contiguous along K
// Both operands contiguous along K, all forms but the first, in the two modes.
constexpr SmallTimes kSmallTimesLines[2][5] = {
    {{}, {1.62, 1.53, 0.00137, 3.1, 0.00146, 0.0, 0.88, 0.89}, {2.91, 1.5, 0.00231, 2.17, 0.00282, 0.0, 0.11, 0.75},
     {1.96, 4.58, 0.00216, 3.46, 0.00191, 0.0, 0.0, 0.73}, {1.93, 2.45, 0.00218, 4.14, 0.00258, 0.0, 0.5, 0.72}},
    {{}, {1.76, 1.37, 0.00104, 2.7, 0.00125, 0.0, 1.15, 0.93}, {3.66, 1.19, 0.00194, 1.2, 0.00193, 0.0, 0.62, 0.62},
     {2.25, 3.95, 0.00164, 2.83, 0.00161, 0.0, 3.0, 0.75}, {1.0, 2.69, 0.00157, 4.13, 0.00249, 0.0, 2.07, 0.83}}};
static_assert(SMALL_32x32 == 0 && SMALL_32x64 == 1 && SMALL_64x64 == 2 && SMALL_64x64_LINES8 == 3 && SMALL_64x64_LINES4 == 4, "the order of the tables");

// The form of the small-tile kernel that beats the kernel the problem would otherwise take by 5 %, or SMALL_NONE.  On 900
// random problems of the storage orders but one it takes 1.5 % (the tiled kernel's problems) and 2.5 % (the others) longer than the best of
// all forms.  Operands whose rows start anywhere, both of them, cost a fifth more, and beyond 16 workgroups of 64 x 64 a compute unit, when
// they no longer come out of the caches, again a third
// (4096 x 5025 x 2048: 200 us, the any-shape kernel 176).  Rows along K of fewer than 16 bytes are fetched byte by byte
// (22 x 275 x 12: 13 us, the any-shape kernel 7.6).  The tiled kernel: rounds of 256 workgroups; where a single round leaves
// half of the compute units idle, a tile has more of the caches to itself (512 x 4400 x 12096 in the FP8 mode: 65 us, 94 on
// 64 x 64 tiles, and 93 by tile_times()).
// Where both operands are contiguous along K that answer stands if it is 32 x 32 (eight waves, the shortest chains of sums); the other
// forms, five in all, are told apart by a table of their own, fitted to every form's time on 2500 random problems (1 .. 4096 x 64 .. 12288
// x 48 .. 12288, ragged ones among them, all output kinds; rows at any place cost a half more, 1.35 beyond 16 workgroups) and on 256 of 32
// to 512 tokens through layers 2048 to 12288 wide: 1.4 % (2.6 % off the tiled kernel) and 0.8 % longer than the best of all, where the
// general table with its three forms takes 2.0 (3.0) and 5.5 %.
// What went to small tiles stays with them (the tiled kernel's one chain of sums is further from the 64-bit result), what did not
// goes over for 8 % (`other` is up to a third too long where 192-wide or mixed tiles are taken).
// us_chosen: the time of what was chosen.
// pinned: one of the three tile sizes, whatever it takes; the forms with 64 x 64 tiles are chosen from all the same, or named by
// FP8_KNOB_SMALL_64.
int choose_small(const GemmArgs& g, bool tiled, double& us_chosen, int pinned)
{
    const double M = (double)g.M, N = (double)g.N, K = (double)g.K;
    auto units = [&](int64_t tm, int64_t tn) { return (double)((g.M + tm - 1) / tm) * (double)((g.N + tn - 1) / tn) / 256.0; };
    const double u64 = units(64, 64);
    double other;
    if (tiled) {
        const TileTimes t = tile_times(g.acc, 2.0 * std::ceil(K / (2 * TILE_K)));
        other = std::min(std::ceil(units(256, 256)) * t.wide, std::ceil(units(256, 128)) * t.narrow);
        if (g.acc == ACC_FP8) other += 1.5;                  // (the fit is that much too short below S = 16)
        if (units(256, 128) < 1.0) {
            const double S = 2.0 * std::ceil(K / (2 * TILE_K)), alone = g.acc == ACC_FP8 ? 8.0 + 0.28 * S : 9.0 + 0.53 * S;
            other = std::min(other, alone + (other - alone) * std::max(0.0, 2.0 * units(256, 128) - 1.0));
        }
    } else {
        other = small_line_us(g);
        if (g.ep.out_kind != OUT_F32 && !g.ep.amax_out) other = std::min(other, 1.1 * std::min(any_us(g, 256), any_us(g, 128)));     // (1.1: their error where a round is short)
    }
    us_chosen = other;
    if (u64 > 32 && pinned == SMALL_NONE) return SMALL_NONE;
    // (what the tiled kernel does not take is computed in the fp16 mode, whatever the flag says)
    const bool lines = !g.transA && g.transB, fp8 = tiled && g.acc == ACC_FP8;
    const bool off_a = !aligned16(g.A) || (g.transA ? g.M : g.K) % 16 != 0, off_b = !aligned16(g.B) || (g.transB ? g.K : g.N) % 16 != 0;
    const double off = off_a && off_b ? (u64 > 16 ? 1.56 : 1.2) : 1.0;
    const double bytewise = g.K < 16 ? 0.35 * K * ((g.transA ? 0 : 1) + (g.transB ? 1 : 0)) : 0.0;
    auto us_of = [&](int f, const SmallTimes& t, double per_k, double places) {
        const double n = f == SMALL_32x32 ? units(32, 32) : f == SMALL_32x64 ? units(32, 64) : u64, full = t.fullest > 0.0 && n <= 4.0 ? n + t.fullest * (std::ceil(n) - n) : n;
        const double waits = std::max(0.0, n - 1.0) * (t.further + ((f == SMALL_64x64 ? g.K % 64 : g.K % 128) ? t.ragged : 0.0));
        return t.ends + places * std::max(t.alone + bytewise + t.alone_k * K, full * (t.each + bytewise + per_k * K) + waits);
    };
    int form = SMALL_NONE;
    double best = pinned == SMALL_NONE ? 0.95 * other : 1e300;
    for (int f = SMALL_32x32; f <= SMALL_64x64; ++f) {
        if (pinned != SMALL_NONE && f != pinned) continue;
        const double us = us_of(f, kSmallTimes[f], lines && f == SMALL_32x32 ? kPerK32Lines : kSmallTimes[f].per_k, off);
        if (us < best) { best = us_chosen = us; form = f; }
    }
    if (!lines || form == SMALL_32x32) return form;
    const double off_lines = off_a && off_b ? (u64 > 16 ? 1.35 : 1.5) : 1.0;
    const int form64 = knob(FP8_KNOB_SMALL_64);
    best = form == SMALL_NONE && pinned == SMALL_NONE ? 0.92 * other : 1e300;
    form = SMALL_NONE;
    for (int f = SMALL_32x64; f <= SMALL_64x64_LINES4; ++f) {
        if (pinned != SMALL_NONE && std::min(f, (int)SMALL_64x64) != pinned) continue;
        if (form64 && f >= SMALL_64x64 && f != SMALL_64x64 + form64 - 1) continue;
        const SmallTimes& t = kSmallTimesLines[fp8 ? 1 : 0][f];
        const double us = us_of(f, t, t.per_k, off_lines);
        if (us < best) { best = us_chosen = us; form = f; }
    }
    return form;
}

}  // namespace

// Which kernel a (non-empty, K > 0) problem takes.  whole: also what it would take without the small tiles (a launch does without: a
// quarter of the host time of the choice).
GemmPlan plan_gemm(const GemmArgs& g, bool whole)
{
    const int64_t M = g.M, N = g.N, K = g.K;
    GemmPlan plan{!force_generic() && mfma_any_takes(g) ? GEMM_MFMA_ANY : GEMM_GENERIC, false, false, 0, SMALL_NONE, false, 0, 1e300};
    // a knob that asks for another form of the kernels keeps the small one out, unless FP8_KNOB_SMALL names a form of it
    const int small = g.splits <= 1 && !force_generic() ? knob(FP8_KNOB_SMALL) : 1;
    const bool small_allowed = small == 0 && !knob(FP8_KNOB_TILE_N) && !knob(FP8_KNOB_GEMM_KERNEL) && !knob(FP8_KNOB_MIXED) && !knob(FP8_KNOB_PERSIST) && knob(FP8_KNOB_TILE_192) != 2;
    const uint64_t ldmax = (uint64_t)(M > N ? (M > K ? M : K) : (N > K ? N : K));
    const bool fits32 = 256 * ldmax < (1ull << 32) && M < (1ll << 31) - TILE_M && N < (1ll << 31) - TILE_N &&
                        K < (1ll << 31) &&
                        // the grid holds one workgroup per tile: counted with the narrow tile, the larger count
                        ((M + TILE_M - 1) / TILE_M) * ((N + TILE_N / 2 - 1) / (TILE_N / 2)) < (1ll << 31);
    // The tiled kernel works on 256 x 256 tiles and clips the last ones: loads of rows / columns
    // beyond the edge are redirected to existing ones and their outputs are not stored.  What it
    // needs: K a multiple of 16 if an operand is contiguous along K (its rows start every K bytes; K is walked in pairs of
    // stages of 64 and a last, partial pair filled up with zeros); 16-byte aligned operands;
    // rows of an N-contiguous B and of an M-contiguous A that start on 16-byte boundaries (N % 16, M % 16).  Rows of C (and a
    // per-column factor vector) may start anywhere (the epilogue's stores go to any address): with
    // B stored N x K any N goes (a vocabulary-sized output layer, weights stored [out, in]).
    // Any K goes where neither operand is contiguous along it (a weight gradient over any number of tokens): what the last stage
    // lacks are whole K-rows, each one load's.  In the fp16 mode, whatever the flag says, and with one factor per operand (those
    // of rows and columns are rounded more often here), so that nothing is less accurate than on the any-shape kernel; what
    // the small tiles, with their shorter chains of sums, took beside that kernel they keep.  Against the any-shape kernel: 4096 x 4096 x 33 43.7 ->
    // 16.8 us, 3648 x 6272 x 100 61.9 -> 25.1, 896 x 12224 x 7259 192 -> 134, 2432 x 8256 x 4489 258 -> 166, 8192 x 12288 x 3333 580 -> 532
    // (beside the any-shape kernel's forms of that time; no product of 47 more than 3 % slower.  The present ones take 16.4 us for the first, the tiled kernel 16.1).
    const bool ragged = K % 16 != 0;
    const int acc = ragged ? (int)ACC_F16 : g.acc;
    const bool c_lines = N % 16 == 0 && aligned16(g.C) && (!g.ep.b_per_col || aligned16(g.ep.sB_dev));
    const bool fast = !force_generic() && !force_mfma_any() && aligned16(g.A) && aligned16(g.B) && fits32 && (!ragged || (g.transA && !g.transB && !g.ep.a_per_row && !g.ep.b_per_col)) &&
                      (g.transB || N % 16 == 0) && (!g.transA || M % 16 == 0);
    if (small_allowed) plan.small = choose_small(g, fast && !ragged, plan.us, SMALL_NONE);
    else if (small >= 2 && tile_count(g, 32) <= 0x7fffffffll) plan.small = choose_small(g, fast && !ragged, plan.us, SMALL_32x32 + small - 2);
    if (!fast) return plan;
    if (!whole && plan.small != SMALL_NONE) {
        plan.kernel = ragged ? GEMM_MFMA_ANY : GEMM_TILED_256;
        return plan;
    }
    // Tile width.  One workgroup per compute unit (256 of them) runs at a time: the width whose rounds
    // of workgroups take less time (4096 x 6144: 384 wide tiles = two rounds, the second half empty, 768
    // narrow ones = three).  The knob FP8_KNOB_TILE_N = 128 | 256 overrides the choice.
    const TileTimes tile = tile_times(acc, 2.0 * (double)((K + 2 * TILE_K - 1) / (2 * TILE_K)));
    const int64_t tiles_m = (M + TILE_M - 1) / TILE_M, wide_cols_all = (N + TILE_N - 1) / TILE_N;
    auto rounds = [&](int64_t tiles) { return (double)((tiles + 255) / 256); };
    const int tn = knob(FP8_KNOB_TILE_N), mk = knob(FP8_KNOB_MIXED), pk = knob(FP8_KNOB_PERSIST), middle_knob = knob(FP8_KNOB_TILE_192);
    const bool narrow = tn ? tn == 128 : rounds(tiles_m * ((N + 127) / 128)) * tile.narrow < rounds(tiles_m * wide_cols_all) * tile.wide;
    plan.kernel = narrow ? GEMM_TILED_128 : GEMM_TILED_256;
    plan.elementwise_stores = !c_lines;
    // Both widths in one launch (gemm_mixed_kernel): the first c tile columns of 256, the rest of N in
    // tiles of 128.  Chosen where a model of the run time says it beats the better single width by 3 %:
    // workgroups are handed to the 256 compute units in order, the wide ones first; a tile takes
    // what tile_times() says, and the change of width costs 3 us and up to 350 / S more, the more the
    // fuller the narrow tiles' last round is (4096 x 6144 over K = 2048 .. 8192, 3001 x 6144 x 2048).  With these
    // figures it pays for long K (4096 x 6144 x 8192: 4 % in the fp16 mode, 7 % in the FP8 mode) and where
    // the wide tiles fill little of their last round (3001 x 6144 x 2048: 3 - 7 %).  Problems of
    // more than 64 rounds are left alone (the last round is then under 2 %).
    // Knob FP8_KNOB_MIXED: 0 = by the model, 1 = never, 2 = wherever it is possible.
    const double S = 2.0 * (double)((K + 2 * TILE_K - 1) / (2 * TILE_K));
    double chosen_us = 1e300;
    // time until the last of Tw wide tiles (tw us each) and then Tn narrow ones ends on 256 units
    const double tnar = tile.narrow;
    auto makespan = [&](int64_t Tw, int64_t Tn, double tw) {
        const int64_t q = Tw / 256, k = Tw % 256;          // k units get q + 1 wide tiles, the others q
        if (Tn == 0) return (double)(q + (k > 0)) * tw;
        double best = 1e300;
        for (int64_t r = 0; r <= Tn; ++r) {                // r narrow tiles on the units that are free first
            const int64_t late = r * tnar >= tw ? (int64_t)((r * tnar - tw) / tnar) : 0;     // and as many as fit on the others
            if ((256 - k) * r + k * late >= Tn) { best = std::max((double)(q + (k > 0)) * tw, (double)q * tw + (double)r * tnar); break; }
        }
        for (int64_t r = 1; r <= Tn; ++r) {                // or the last one ends on a unit that had q + 1 wide tiles
            const int64_t early = (int64_t)((tw + r * tnar) / tnar);
            if (k * r + (256 - k) * early >= Tn) { best = std::min(best, (double)(q + 1) * tw + (double)r * tnar); break; }
            if ((double)(q + 1) * tw + (double)r * tnar >= best) break;
        }
        return best;
    };
    const bool few_rounds = plan.small == SMALL_NONE && g.splits <= 1 && tiles_m * wide_cols_all <= 64 * 256;
    if (few_rounds) chosen_us = std::min(makespan(tiles_m * wide_cols_all, 0, tile.wide), makespan(0, tiles_m * ((N + 127) / 128), tile.wide));
    if (!tn && mk != 1 && few_rounds && N > TILE_N) {
        const double uniform = chosen_us;
        double best = 1e300;
        int64_t best_c = 0;
        for (int64_t c = 1; c * TILE_N < N; ++c) {
            const int64_t Tn = tiles_m * ((N - c * TILE_N + 127) / 128);
            const double change = 3.0 + 350.0 / S * (double)(Tn % 256 ? Tn % 256 : 256) / 256.0;
            const double t = makespan(tiles_m * c, Tn, tile.wide) + change;
            if (t < best) { best = t; best_c = c; }
        }
        if (best_c > 0 && (mk == 2 || best < 0.97 * uniform)) {
            plan.kernel = GEMM_TILED_MIXED;
            plan.wide_cols = (int)best_c;
            chosen_us = best;
        }
    }
    // The persistent form of the narrow tile (one workgroup per compute unit walks its tiles as one K
    // loop, see gemm_tiled.hip): for problems of more than one round of tiles without edge tiles, with
    // per-tensor factors and an fp32 / bf16 output.  It hides every tile's first loads and sends the
    // outputs straight from the registers, but its workgroups cannot even out their speeds over the
    // tiles as separately scheduled ones do.  Measured on 4096 x 6144 (768 tiles): with fp32 outputs
    // 3 - 6 % faster up to K = 4096 in both accumulation modes (the LDS turn of an fp32 tile takes two
    // passes); with bf16 outputs 2 % faster around K = 2048 in the fp16 mode, slower in the FP8 mode;
    // 1 - 2 % slower at K = 8192 throughout.  Knob FP8_KNOB_PERSIST: 0 = where it pays (below),
    // 1 = never, 2 = wherever it is possible.
    const int64_t tiles = tiles_m * ((N + 127) / 128);
    const bool possible = plan.kernel == GEMM_TILED_128 && c_lines && M % TILE_M == 0 && N % 128 == 0 && K % (2 * TILE_K) == 0 && K >= 8 * TILE_K &&
                          !g.ep.a_per_row && !g.ep.b_per_col && g.ep.out_kind <= OUT_BF16 && !g.ep.amax_out && g.splits <= 1;
    const bool pays = tiles > 256 && (g.ep.out_kind == OUT_F32 ? K <= 64 * TILE_K
                                                               : acc == ACC_F16 && K >= 16 * TILE_K && K <= 32 * TILE_K);
    plan.persistent = possible && plan.small == SMALL_NONE && pk != 1 && (pk == 2 || pays);
    // Tiles of 256 x 192, alone or with 128-wide ones behind them: where the same model says that they beat the choice so
    // far by 3 % (4096 x 6144 x 2048: 512 tiles = two full rounds, 84 us against 93 for 768 narrow ones; 3001 x 6144 x 2048:
    // 252 of them and 204 narrow ones, 85 us against 90 for 384 of them and 94 for 252 wide and 72 narrow ones).  Of 70 products in the
    // range where it decides, 19 took them, and no other would have gained more than 2 %.  240 random products that take them, all
    // storage orders and outputs: 1.10 times as fast in the mean (1.05 to 1.13 by order and mode), 0.93 to 1.29; two of them more than 3 %
    // slower, FP8 mode with fp32 outputs.
    // fp32 outputs that the persistent narrow form takes stay there (4096 x 6144 x 1024: 57 us, here 59).
    // Knob FP8_KNOB_TILE_192: 0 = by the model, 1 = never, 2 = always (with FP8_KNOB_MIXED = 2: for half of the columns, 128-wide ones behind).
    if (middle_knob == 2) {
        plan.middle = true;
        plan.middle_cols = mk == 2 && N > 192 ? (int)((N + 191) / 384) : 0;
    } else if (middle_knob == 0 && !tn && !mk && !pk && few_rounds && !(plan.persistent && g.ep.out_kind == OUT_F32)) {
        double best = makespan(tiles_m * ((N + 191) / 192), 0, tile.middle);
        for (int64_t units = 256; units / tiles_m * 192 < N; units += 256) {     // as many columns as whole rounds hold
            const int64_t c = units / tiles_m;
            if (c == 0) continue;
            const int64_t Tn = tiles_m * ((N - c * 192 + 127) / 128);
            const double t = makespan(tiles_m * c, Tn, tile.middle) + 2.0 + 100.0 / S * (double)(Tn % 256 ? Tn % 256 : 256) / 256.0;
            if (t < 0.97 * best) { best = t; plan.middle_cols = (int)c; }
        }
        plan.middle = best < 0.97 * chosen_us;
    }
    return plan;
}

// ---- the matrix-core kernel for any shape (gemm_mfma_any.hip) ------------------------------------
bool mfma_any_takes(const GemmArgs& g)
{
    return g.M > 0 && g.N > 0 && g.K > 0 && tile_count(g, 128) <= 0x7fffffffll && (mfma_any_width(g) || tile_count(g, 64) <= 0x7fffffffll);
}

// The narrower tile unless the wider one saves 6 %, the model's error; FP8_KNOB_TILE_N forces either.  Not for the kernel's tiles: an operand
// contiguous along M / N with rows of fewer than 16 bytes, offsets within a tile's stage beyond 32 bits.
int mfma_any_width(const GemmArgs& g)
{
    if (g.M >= (1 << 26) || g.N >= (1 << 26) || (g.transA && g.M < 16) || (!g.transB && g.N < 16)) return 0;
    const int forced = knob(FP8_KNOB_TILE_N);
    if (forced) return forced;
    return any_us(g, 256) < 0.94 * any_us(g, 128) ? 256 : 128;
}

namespace {

int launch_small(const GemmArgs& g, int form)
{
    typedef int (*small_fn)(const GemmArgs&, int);
    static const small_fn table[4] = {FP8MM_SMALL_NAME(0), FP8MM_SMALL_NAME(1), FP8MM_SMALL_NAME(2), FP8MM_SMALL_NAME(3)};
    return table[(g.transA ? 2 : 0) + (g.transB ? 1 : 0)](g, form);
}

}  // namespace

int launch_mfma_any(const GemmArgs& g)
{
    typedef int (*any_fn)(const GemmArgs&, int);
    static const any_fn table[4] = {FP8MM_ANY_NAME(0), FP8MM_ANY_NAME(1), FP8MM_ANY_NAME(2), FP8MM_ANY_NAME(3)};
    if (const int width = mfma_any_width(g)) return table[(g.transA ? 2 : 0) + (g.transB ? 1 : 0)](g, width);
    GemmArgs gs = g;
    gs.acc = ACC_F16;
    return launch_small(gs, SMALL_64x64);
}

// Chunks of 128 of both operands in LDS (rows of 128 + 16 bytes, or of 32 + 16), at least the waves' sums.
int scaled_gemm_small_lds(const GemmArgs& g)
{
    const int chunks = (int)((g.K + 127) / 128), slabs = chunks * ((g.transA ? 128 * 48 : 32 * 144) + (g.transB ? 32 * 144 : 128 * 48));
    return std::max(slabs, 8 * 32 * 36 * 4);
}

namespace {

bool overlap(const void* p, int64_t np, const void* q, int64_t nq) { return (const char*)p < (const char*)q + nq && (const char*)q < (const char*)p + np; }

// Which problems one launch takes: those of 32 x 32 tiles, at most one a compute unit (256: a workgroup waits for the maxima of others, which
// should be running), rows and columns of up to 2048 bytes (a thread's registers) and, of all tiles together, less than 192 KB along K: they are read and
// rounded once per tile.  90 random products, amax + cast and product apart / together: 61 x 64 x 168 of fp32 9.9 / 6.7 us, 163 x 24 x 656 of bf16
// 11.1 / 9.6, 693 x 304 x 408 (180 KB) 12.1 / 11.1, but 308 x 704 x 824 (362 KB) 12.6 / 13.3; geometric mean 1.37.  As graph nodes, which have no host time to
// save, 187 products below the line gain 1.17 in the geometric mean (calls 1.31); of 11 from there to 288 KB nine lose (0.95 in the
// mean; 512 x 480 x 512 of bf16 10.1 / 11.1, 616 x 248 x 816 11.6 / 12.6), while calls gain 1.06.
// Where rows in memory end inside a vector, K of up to 1024 bytes: 38 such products 1.34 in the geometric mean, least 1.11 (graph nodes 1.19, 0.98;
// 34 x 260 x 87 of fp32 11.6 / 6.8, 41 x 575 x 424 of bf16 11.2 / 9.3), but of 6 with a longer K all but one lost as graph nodes
// (78 x 54 x 579 of bf16 9.9 / 11.1, 674 x 261 x 274 of fp32 9.6 / 11.8; geometric mean 0.94).
// And not many tiles: every workgroup reads all maxima, and the more of them there are the longer the exchange takes (20 tiles of a short K 6.5 us, 90 7.0, 140 8, 240
// 9 - 10), while the launches apart grow by less.  68 products of 100 to 256 tiles, apart / together: beyond 200 tiles all 10 lost as graph nodes and 5 as calls (736 x 344 x 16 of fp32
// 7.9 / 9.3 and 8.5 / 9.4 us; 0.93 and 0.99 in the mean), up to there 29 gain 1.06 and 1.13, no call lost.  An operand contiguous along K whose FP8 rows begin anywhere costs the
// product apart 1 - 3 us: 235 tiles there (20 gain 1.25, none lost; 247 tiles 9.2 / 9.9).  K of up to 16 that neither operand is contiguous along is
// the fastest apart: 64 tiles (20 tiles 7.7 / 6.5; 6 from 110 on all lost, 864 x 288 x 8 7.7 / 9.8).
// Rows in memory of at least a vector; operands that share no memory with an output (a tile is written while others
// are still being loaded).
// (all but the tiles, which take longer to find out)
bool scaled_gemm_small_takes(const GemmArgs& g, const void* a, const void* b, int in_dtype)
{
    const int64_t esz = in_dtype == FP8_F32 ? 4 : 2, pv = 16 / esz;
    const bool along_k = !g.transA || g.transB;
    const int most = along_k && g.K % 16 != 0 ? 235 : !along_k && g.K <= 16 ? 64 : 200;
    if (g.K * esz > kScaledSmallRow || tile_count(g, 32) > std::min(most, compute_units())) return false;
    if (cast_path() != kCastCvt || tile_count(g, 32) * g.K * esz >= kScaledSmallBytes) return false;
    const bool ragged = (g.transA ? g.M : g.K) % pv || (g.transB ? g.K : g.N) % pv;
    if (ragged && g.K * esz > kScaledSmallRow / 2) return false;
    if ((g.transA ? g.M : g.K) < pv || (g.transB ? g.K : g.N) < pv || scaled_gemm_small_lds(g) > kScaledSmallLds) return false;
    const int64_t na = g.M * g.K, nb = g.K * g.N, nc = g.M * g.N * out_elem_size(g.ep.out_kind);
    for (auto [x, n] : {std::pair<const void*, int64_t>{a, na * esz}, {b, nb * esz}})
        if (overlap(x, n, g.C, nc) || overlap(x, n, g.A, na) || overlap(x, n, g.B, nb)) return false;
    return true;
}

}  // namespace

int launch_scaled_gemm_small(const GemmArgs& g, const void* a, const void* b, int in_dtype, float* amax_out, float* scale_out, void* workspace, bool& took,
                             std::optional<GemmPlan>& plan)
{
    typedef int (*scaled_fn)(const GemmArgs&, const void*, const void*, int, float*, float*, void*);
    static const scaled_fn table[4] = {FP8MM_SCALED_NAME(0), FP8MM_SCALED_NAME(1), FP8MM_SCALED_NAME(2), FP8MM_SCALED_NAME(3)};
    took = false;
    if (g.M == 0 || g.N == 0 || g.K == 0 || !scaled_gemm_small_takes(g, a, b, in_dtype)) return FP8_OK;
    plan = plan_gemm(g, false);
    if (plan->small != SMALL_32x32) return FP8_OK;
    took = true;
    GemmArgs gs = g;
    if (plan->kernel == GEMM_MFMA_ANY) gs.acc = ACC_F16;      // as launch_gemm
    return table[(g.transA ? 2 : 0) + (g.transB ? 1 : 0)](gs, a, b, in_dtype, amax_out, scale_out, workspace);
}

int launch_tiled(const GemmArgs& g)
{
    typedef int (*tiled_fn)(const GemmArgs&);
    static const tiled_fn table[4][2] = {
        {FP8MM_TILED_NAME(0, 0), FP8MM_TILED_NAME(0, 1)}, {FP8MM_TILED_NAME(1, 0), FP8MM_TILED_NAME(1, 1)},
        {FP8MM_TILED_NAME(2, 0), FP8MM_TILED_NAME(2, 1)}, {FP8MM_TILED_NAME(3, 0), FP8MM_TILED_NAME(3, 1)}};
    return table[(g.transA ? 2 : 0) + (g.transB ? 1 : 0)][g.acc == ACC_FP8 ? 1 : 0](g);
}

int gemm_form(const GemmArgs& g)
{
    static_assert(FP8_FORM_SMALL_64x64_LINES4 - FP8_FORM_SMALL_32x32 == SMALL_64x64_LINES4, "the order of the forms");
    const GemmPlan plan = plan_gemm(g, false);
    if (plan.small != SMALL_NONE) return FP8_FORM_SMALL_32x32 + plan.small;
    if (plan.kernel == GEMM_GENERIC) return FP8_FORM_FMA;
    if (plan.kernel == GEMM_MFMA_ANY) {
        const int width = mfma_any_width(g);
        return width == 256 ? FP8_FORM_ANY_256 : width ? FP8_FORM_ANY_128 : FP8_FORM_SMALL_64x64;
    }
    if (plan.middle) return plan.middle_cols > 0 ? FP8_FORM_TILED_192_128 : FP8_FORM_TILED_192;
    if (plan.kernel == GEMM_TILED_MIXED) return FP8_FORM_TILED_256_128;
    if (plan.kernel == GEMM_TILED_256) return FP8_FORM_TILED_256;
    return plan.persistent ? FP8_FORM_TILED_128_PERSISTENT : FP8_FORM_TILED_128;
}

int launch_gemm(const GemmArgs& g, const GemmPlan* known)
{
    const int64_t M = g.M, N = g.N, K = g.K;
    if (g.ep.amax_out) {                                     // written, not accumulated
        enqueue(zero_cell_kernel, dim3(1), dim3(1), 0, g.stream, (unsigned*)g.ep.amax_out);
        if (M == 0 || N == 0) return check_launch("gemm (amax init)");
    }
    if (M == 0 || N == 0) return FP8_OK;
    if (K == 0) {                                            // empty sums: every output is +0
        const size_t nbytes = (size_t)M * (size_t)N * (size_t)out_elem_size(g.ep.out_kind);
        enqueue(zero_fill_kernel, dim3(1024), dim3(256), 0, g.stream, (unsigned char*)g.C, nbytes);
        return check_launch("gemm (K = 0 fill)");
    }
    const GemmPlan plan = known ? *known : plan_gemm(g, false);
    if (plan.small != SMALL_NONE) {
        GemmArgs gs = g;
        if (plan.kernel == GEMM_MFMA_ANY) gs.acc = ACC_F16;  // as the any-shape kernel computes these problems
        return launch_small(gs, plan.small);
    }
    if (plan.kernel == GEMM_MFMA_ANY) return launch_mfma_any(g);
    if (plan.kernel != GEMM_GENERIC) {
        GemmArgs gt = g;
        if (K % 16 != 0) gt.acc = ACC_F16;                   // see plan_gemm
        gt.tile_n = plan.middle ? 192 : plan.kernel == GEMM_TILED_128 ? 128 : 256;
        gt.wide_cols = plan.middle ? plan.middle_cols : plan.kernel == GEMM_TILED_MIXED ? plan.wide_cols : 0;
        gt.persist = plan.persistent && !plan.middle;
        gt.splits = 1;
        return launch_tiled(gt);
    }
    if (g.fmtA == FP8_E4M3)
        return g.fmtB == FP8_E4M3 ? launch_generic<FP8_E4M3, FP8_E4M3>(g) : launch_generic<FP8_E4M3, FP8_E5M2>(g);
    return g.fmtB == FP8_E4M3 ? launch_generic<FP8_E5M2, FP8_E4M3>(g) : launch_generic<FP8_E5M2, FP8_E5M2>(g);
}

}  // namespace fp8mm
