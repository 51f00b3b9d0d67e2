// Matrix-core GEMM for any shape and any alignment, for gfx950 (MI355X).
//
//   c[M x N] = (op(A)[M x K] x op(B)[K x N]) / (sA sB),   D = cast_out(c)
//
// The tiled kernel (gemm_tiled.hip) fills its LDS with direct global->LDS loads of aligned 16-byte
// chunks and therefore wants operand rows that start on 16-byte boundaries.  This kernel serves everything else (an odd K of an
// operand that is contiguous along it, an odd leading dimension such as a vocabulary size with the weight stored [in, out],
// operands at any address) with the tiled kernel's products: bytes in LDS as they lie in memory, fragments widened in registers
// under the matrix instructions, v_mfma_f32_32x32x16_f16 with fp32 accumulation, the sums in the same order (bit-identical
// results where both take a problem), so the same error bound holds (arXiv 2209.05433, Section 2: FP8 operands,
// single-precision accumulation, factors taken out once per output).  The loads go through registers, where a piece may start
// at any address:
//   - 256 x 64 NB output tiles (NB = 4 or 2), four waves of 128 x 32 NB, one workgroup per compute unit;
//   - a step multiplies one stage of 64 along K.  Meanwhile a thread writes the 4 + NB vectors of 16 bytes that it
//     requested a step ago to LDS and requests the next ones into the registers that this frees: a load has a whole
//     step to arrive, and no more than 4 + NB of them hold registers;
//   - an operand that is contiguous along M / N is staged one stage (64 K-rows) a step, two stages ahead of the products; one that is
//     contiguous along K half of the rows of a pair of stages, so that its rows are asked for in pieces of 128 bytes, a line
//     at a time: two slabs of either kind, 48 to 128 KB;
//   - tiles that lie inside C walk the stages inside K with one register of offsets per operand and no tests (526 instructions
//     for 128 matrix instructions, no register spilled or moved); at the edges a piece that is not wholly there comes
//     from the zero chunk or is the row's last 16 bytes, shifted when it is written.
// Over a long K bound by the matrix cores at the clock they hold (8192 x 50257 x 12288: busy 73 % of the cycles, at 1.74 GHz; 9 % of the waves' time at
// s_waitcnt, LDS busy 19 %), over a short one by the starts and ends of the tiles (4096 x 50257 x 2048: 53 % at 1.97 GHz; a tile's ends are 8.5 of 58 us, and the last of
// 13 rounds has 80 tiles).  Forced onto a product that the tiled kernel takes, it needs 1.06 - 1.09 of its time (8192 x 50304 x 6144).  The forms before it widened on the way into LDS, which had to carry twice the bytes, and the smaller of them
// stored its outputs one by one.  256 x 256 tile: 4096 x 50257 x 2048 882 -> 765 us, 8192 x 50257 x 12288 9083 -> 7849,
// 8192 x 12288 x 4095 (both contiguous along K) 884 -> 694, 5000 x 5001 x 5001 with A stored K x M 624 -> 274;
// 256 x 128: 4673 x 4573 x 1057 147 -> 72, 1307 x 12288 x 4405 to E4M3 256 -> 223.
//
// This file is compiled once per pair of storage orders: -DFP8MM_LAYOUT.
#include "gemm_epilogue.hpp"
#include "gemm_slabs.hpp"

#include <atomic>
#include <type_traits>

namespace fp8mm {
namespace {

// Sixteen zero bytes in device memory, never written: what stands in for a piece beyond the end of K.
__device__ __attribute__((aligned(16))) uint8_t g_any_zero_chunk[16];

constexpr int FGROUP = 8;               // tile rows per band of the tile order

// Workgroup id -> tile.  Ids go round-robin over the 8 XCDs (each with its own L2); XCD x gets one
// contiguous run of the order below, so that the tiles it works on at a time share a few row slabs
// of A and column slabs of B in its L2 (dealt out id by id, every XCD streamed all of B once per
// band: 47 GB of L2 fills for 0.7 GB of operands, measured).  Order: bands of FGROUP tile rows,
// down the rows of a band first, then to the next tile column.
__device__ __forceinline__ void tile_of(int64_t bid, int64_t tiles_m, int64_t tiles_n, int64_t& tm, int64_t& tn)
{
    const int64_t total = tiles_m * tiles_n;
    const int64_t x = bid % 8, idx = bid / 8, base = total / 8, rem = total % 8;
    const int64_t p = x * base + (x < rem ? x : rem) + idx;
    const int64_t band_tiles = FGROUP * tiles_n;
    const int64_t band = p / band_tiles, q = p - band * band_tiles;
    const int64_t rows = tiles_m - band * FGROUP < FGROUP ? tiles_m - band * FGROUP : FGROUP;
    tm = band * FGROUP + q % rows;
    tn = q / rows;
}

template <bool KC, int EXT>
struct Staged {
    static constexpr int NV = EXT / 64;                   // vectors per thread and step
    static constexpr int CH = KC ? 8 : EXT / 16;          // lanes that share a row
    static constexpr int ROWS = 256 / CH;                 // rows between two vectors of a thread
    static constexpr int SLAB = KC ? EXT * 128 : 64 * EXT;
    const uint8_t* base;                                  // of the operand
    const uint8_t* tile;                                  // KC: first row of the tile, MC: its first column
    int64_t ld, K;                                        // bytes between rows; K
    int64_t last;                                         // KC: last row of the operand, counted from the tile's first
    int row, at;                                          // of the thread's first vector: row (MC: K-row), byte in it
    int back;                                             // MC: bytes that the thread's column is moved back to stay in the row
    unsigned off;                                         // row * ld + at
    unsigned lds;                                         // where the first vector goes in the first slab

    __device__ __forceinline__ void setup(const uint8_t* base_, int64_t ext, int64_t K_, int64_t t0, unsigned region, int tid)
    {
        base = base_;
        K = K_;
        ld = KC ? K : ext;
        tile = KC ? base + t0 * K : base + t0;
        last = ext - 1 - t0;
        row = tid / CH;
        at = (tid % CH) * 16;
        off = (unsigned)row * (unsigned)ld + (unsigned)at;
        // (a column wholly outside reads the row's last 16 bytes: its products are not stored)
        back = !KC && t0 + at + 16 > ext ? (int)(t0 + at + 16 - ext) : 0;
        if (KC) lds = region + row * 128 + (((tid % CH) ^ swz_kc(row)) * 16);
        else lds = region + row * EXT + mc_pos<CH>(tid % CH, row) * 16;
    }
    // Vector v of load set `set`: KC: half set % 2 of the rows of pair set / 2; MC: stage `set`.
    __device__ __forceinline__ u32x4 load(int64_t set, int v) const             // wholly inside the operand
    {
        const int64_t k = KC ? (set >> 1) * 128 : set * 64 * ld, r = KC ? (set & 1) * (EXT / 2) + v * ROWS : v * ROWS;
        return *(const u32x4_any*)(tile + k + r * ld + off);
    }
    __device__ __forceinline__ u32x4 load_edge(int64_t set, int v) const        // see write; KC: K >= 16 or beyond it, MC: ext >= 16
    {
        const uint8_t* p;
        if (KC) {
            const int64_t k = (set >> 1) * 128 + at, r = (set & 1) * (EXT / 2) + v * ROWS + row;
            p = k >= K ? g_any_zero_chunk : tile + (r < last ? r : last) * ld + (k + 16 <= K ? k : K - 16);
        } else {
            const int64_t k = set * 64 + v * ROWS + row;
            p = k >= K ? g_any_zero_chunk : tile + k * ld + at - back;
        }
        return *(const u32x4_any*)p;
    }
    // The first sets: as load_edge, and any K.  (Of a row shorter than a vector the last 16 bytes up to its end, which begin in the
    // rows before it and are shifted out like any others; byte by byte where the operand begins behind them.)
    __device__ __forceinline__ u32x4 load_first(int64_t set, int v) const
    {
        if (KC && K < 16 && (set >> 1) == 0 && at == 0) {
            const int64_t r = (set & 1) * (EXT / 2) + v * ROWS + row;
            const uint8_t* p = tile + (r < last ? r : last) * ld;
            return p + K - base >= 16 ? *(const u32x4_any*)(p + K - 16) : load_short(p, (int)K);
        }
        return load_edge(set, v);
    }
    // The vector into the slab of its set.  EDGE: it came from load_edge.
    template <bool EDGE>
    __device__ __forceinline__ void write(uint8_t* smem, int64_t set, int v, u32x4 x) const
    {
        if (EDGE) {
            const int64_t beyond = KC ? (set >> 1) * 128 + at + 16 - K : back;
            x = drop_bytes(x, beyond > 0 && beyond < 16 ? (int)beyond : 0);
        }
        const unsigned to = lds + (KC ? (unsigned)((set >> 1) & 1) * SLAB + (unsigned)((set & 1) * (EXT / 2) + v * ROWS) * 128
                                      : (unsigned)(set & 1) * SLAB + (unsigned)(v * ROWS) * EXT);
        *LDS_PTR(u32x4, smem + to) = x;
    }
};

template <bool A_KC, bool B_KC, int NB>
constexpr int any_lds()
{
    const int slabs = 2 * (Staged<A_KC, 256>::SLAB + Staged<B_KC, 64 * NB>::SLAB);
    return slabs > EP_AMAX + 1024 ? slabs : EP_AMAX + 1024;
}

template <int FMT_A, int FMT_B, bool A_KC, bool B_KC, int NB>
__global__ __launch_bounds__(256, 1) void gemm_mfma_any_kernel(
    const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, void* __restrict__ C,
    int64_t M, int64_t N, int64_t K, EpilogueArgs ep)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    typedef Staged<A_KC, 256> StagedA;
    typedef Staged<B_KC, 64 * NB> StagedB;
    constexpr int BN = 64 * NB, P = 2 * NB;               // tile width; parts of a step
    constexpr unsigned B_REGION = 2 * StagedA::SLAB;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int wm = w >> 1, wn = w & 1;
    int64_t tm, tn;
    tile_of(blockIdx.x, (M + 255) / 256, (N + BN - 1) / BN, tm, tn);
    const int64_t m0 = tm * 256, n0 = tn * BN;
    const int64_t KT = 2 * ((K + 127) / 128);             // stages, the last of them possibly zeros

    StagedA a; StagedB b;
    a.setup(A, M, K, m0, 0, tid);
    b.setup(B, N, K, n0, B_REGION, tid);
    const unsigned rd_a = fragment_start<A_KC, 256>(0, wm, l), rd_b = fragment_start<B_KC, BN>(B_REGION, wn, l);

    v16f acc[NB][4];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // The products of a part and the widening for it, a part ahead: see the tiled kernel.
    v8h a16[2][4], b16[2][2];
    auto convert = [&](int j, v8i (&af)[4], v8i (&bf)[NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int s = (2 * j + i) / NB, nb = (2 * j + i) % NB;
            b16[j & 1][i] = widen8<FMT_B>(bf[nb][2 * s], bf[nb][2 * s + 1]);
        }
        if ((2 * j) % NB == 0) {
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) a16[(2 * j / NB) & 1][mb] = widen8<FMT_A>(af[mb][2 * (2 * j / NB)], af[mb][2 * (2 * j / NB) + 1]);
        }
    };
    auto compute = [&](int j) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int s = (2 * j + i) / NB, nb = (2 * j + i) % NB;
#pragma unroll
            for (int mb = 0; mb < 4; ++mb)
                acc[nb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b16[j & 1][i], a16[s & 1][mb], acc[nb][mb], 0, 0, 0);
        }
    };
    auto read_both = [&](int parity, int pair_slot, int j, v8i (&af)[4], v8i (&bf)[NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int ra = j * 8 / P; ra < (j + 1) * 8 / P; ++ra) read_part<A_KC, 256, 2>(smem, rd_a, parity, pair_slot, ra & 3, ra >> 2, af);
        read_part<B_KC, BN, 2>(smem, rd_b, parity, pair_slot, j % NB, j / NB, bf);
    };

    // Load sets: step s writes set s + 2 of an operand contiguous along M / N (a stage), set s + 3 of one contiguous along K (a
    // half pair; sets 0 .. 2 are the first pair and half of the second), and requests the set after it.
    u32x4 xa[StagedA::NV], xb[StagedB::NV];
    constexpr int AHEAD_A = A_KC ? 3 : 2, AHEAD_B = B_KC ? 3 : 2;
    {
        u32x4 fa[AHEAD_A][StagedA::NV], fb[AHEAD_B][StagedB::NV];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
            for (int v = 0; v < StagedA::NV; ++v)
                if (q < AHEAD_A) fa[q][v] = a.load_first(q, v);
#pragma unroll
            for (int v = 0; v < StagedB::NV; ++v)
                if (q < AHEAD_B) fb[q][v] = b.load_first(q, v);
        }
#pragma unroll
        for (int v = 0; v < StagedA::NV; ++v) xa[v] = a.load_edge(AHEAD_A, v);
#pragma unroll
        for (int v = 0; v < StagedB::NV; ++v) xb[v] = b.load_edge(AHEAD_B, v);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
            for (int v = 0; v < StagedA::NV; ++v)
                if (q < AHEAD_A) a.template write<true>(smem, q, v, fa[q][v]);
#pragma unroll
            for (int v = 0; v < StagedB::NV; ++v)
                if (q < AHEAD_B) b.template write<true>(smem, q, v, fb[q][v]);
        }
    }
    // All of the wave's LDS accesses have completed, then all of the workgroup's.  (Loads stay in flight.)
    auto barrier = [&]() __attribute__((always_inline)) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
    };
    v8i af0[4], bf0[NB], af1[4], bf1[NB];
    barrier();
#pragma unroll
    for (int j = 0; j < P; ++j) read_both(0, 0, j, af0, bf0);
    convert(0, af0, bf0);

    // Step s multiplies stage s, whose fragments are in (af, bf), and reads those of stage s + 1.  Behind its barrier stage
    // s + 1 is complete in LDS, and nobody reads the slab that stage s (or the pair before that of stage s + 1) lay in.
    // EDGE: the pieces of this step may lie over an edge.  The last two steps stage nothing.
    constexpr int READS = 8 / P * (A_KC ? 1 : 2) + (B_KC ? 1 : 2), VECTORS = StagedA::NV + StagedB::NV;
    auto step = [&](auto edge_tag, auto stage_tag, int64_t s, int odd, v8i (&af)[4], v8i (&bf)[NB], v8i (&af_n)[4], v8i (&bf_n)[NB]) __attribute__((always_inline)) {
        constexpr bool EDGE = decltype(edge_tag)::value, STAGE = decltype(stage_tag)::value;
        barrier();
        const int pair_slot = (int)((s + 1) >> 1) & 1;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            if (STAGE) {
#pragma unroll
                for (int i = 0; i < VECTORS; ++i) {
                    if (i * P / VECTORS != j) continue;
                    // A's and B's vectors in turn, as long as B has some
                    const bool of_a = i >= 2 * StagedB::NV || i % 2 == 0;
                    const int v = i >= 2 * StagedB::NV ? i - StagedB::NV : i / 2;
                    if (of_a) {
                        a.template write<EDGE>(smem, s + AHEAD_A, v, xa[v]);
                        xa[v] = EDGE ? a.load_edge(s + AHEAD_A + 1, v) : a.load(s + AHEAD_A + 1, v);
                    } else {
                        b.template write<EDGE>(smem, s + AHEAD_B, v, xb[v]);
                        xb[v] = EDGE ? b.load_edge(s + AHEAD_B + 1, v) : b.load(s + AHEAD_B + 1, v);
                    }
                }
            }
            read_both(odd ^ 1, pair_slot, j, af_n, bf_n);
            compute(j);
            if (j + 1 < P) convert(j + 1, af, bf); else convert(0, af_n, bf_n);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                    // MFMA
                if (i < READS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // LDS read
                if (STAGE && i >= 6) {
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);                // LDS write
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                // load
                }
                __builtin_amdgcn_sched_group_barrier(0x002, EDGE ? 6 : 3, 0);         // widening for the next part
            }
            __builtin_amdgcn_sched_barrier(0);        // nothing drifts into another part (register pressure)
        }
    };
    const std::integral_constant<bool, true> yes;
    const std::integral_constant<bool, false> no;
    // stages inside K of a tile inside C: the two steps of a trip request stages up to s + 5
    int64_t s = 0;
    const int64_t inside = (m0 + 256 <= M && n0 + BN <= N) && (A_KC ? K : M) < (1 << 26) && (B_KC ? K : N) < (1 << 26) ? K / 64 : 0;
    for (; s + 6 <= inside; s += 2) {
        step(no, yes, s, 0, af0, bf0, af1, bf1);
        step(no, yes, s + 1, 1, af1, bf1, af0, bf0);
    }
    for (; s + 2 < KT; s += 2) {
        step(yes, yes, s, 0, af0, bf0, af1, bf1);
        step(yes, yes, s + 1, 1, af1, bf1, af0, bf0);
    }
    step(no, no, s, 0, af0, bf0, af1, bf1);
#pragma unroll
    for (int j = 0; j < P; ++j) {
        compute(j);
        if (j + 1 < P) convert(j + 1, af1, bf1);
    }
    __syncthreads();                                  // every wave is done with the slabs
    store_tile<NB, true>(acc, smem, ep, C, (int)M, (int)N, (int)m0, (int)n0, w);
}

template <int FA, int FB, bool A_KC, bool B_KC, int NB>
int launch_tile(const GemmArgs& g)
{
    // more dynamic LDS than the default limit: raised once per device
    constexpr int LDS = any_lds<A_KC, B_KC, NB>();
    static std::atomic<unsigned long long> attr_set{0ull};
    auto kern = gemm_mfma_any_kernel<FA, FB, A_KC, B_KC, NB>;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(FP8_ERR_DEVICE, "hipGetDevice failed");
    const unsigned long long bit = 1ull << (dev & 63);
    if (dev >= 64 || !(attr_set.load(std::memory_order_relaxed) & bit)) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess)
            return fail(FP8_ERR_DEVICE, "hipFuncSetAttribute(LDS=%d): %s", LDS, hipGetErrorString(e));
        if (dev < 64) attr_set.fetch_or(bit, std::memory_order_relaxed);
    }
    const int64_t tiles = ((g.M + 255) / 256) * ((g.N + 64 * NB - 1) / (64 * NB));
    enqueue(kern, dim3((unsigned)tiles), dim3(256), LDS, g.stream, g.A, g.B, g.C, g.M, g.N, g.K, g.ep);
    return check_launch("gemm (matrix-core kernel for any shape)");
}

template <int FA, int FB, bool A_KC, bool B_KC>
int launch_one(const GemmArgs& g, int width)
{
    return width == 256 ? launch_tile<FA, FB, A_KC, B_KC, 4>(g) : launch_tile<FA, FB, A_KC, B_KC, 2>(g);
}

}  // namespace

#if !defined(FP8MM_LAYOUT)
#error "compile with -DFP8MM_LAYOUT=0..3 (2 * transA + transB)"
#endif

// This file is compiled once per pair of storage orders (-DFP8MM_LAYOUT): A stored M x K is
// K-contiguous, B stored N x K (transB) is K-contiguous.
int FP8MM_ANY_NAME(FP8MM_LAYOUT)(const GemmArgs& g, int width)
{
    constexpr bool A_KC = (FP8MM_LAYOUT & 2) == 0, B_KC = (FP8MM_LAYOUT & 1) != 0;
    if (g.fmtA == FP8_E4M3)
        return g.fmtB == FP8_E4M3 ? launch_one<FP8_E4M3, FP8_E4M3, A_KC, B_KC>(g, width) : launch_one<FP8_E4M3, FP8_E5M2, A_KC, B_KC>(g, width);
    return g.fmtB == FP8_E4M3 ? launch_one<FP8_E5M2, FP8_E4M3, A_KC, B_KC>(g, width) : launch_one<FP8_E5M2, FP8_E5M2, A_KC, B_KC>(g, width);
}

}  // namespace fp8mm
