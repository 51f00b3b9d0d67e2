// The whole scaled product (amax, factor and cast of both operands, FP8 product) of a small problem in ONE launch, for gfx950 (MI355X).
//
// A 256 x 256 product as two launches (amax + cast, small tiles) takes 8.9 us, of which the products are a few hundred
// nanoseconds: each launch begins with loads that take a microsecond, the first ends in an exchange of maxima between its
// workgroups, and the second waits for the first.  Here a workgroup of 8 waves owns a 32 x 32 output tile and loads the 32 rows of op(A) and the 32
// columns of op(B) that it needs in their wide type, all of them at once, into registers:
//   - the workgroups of the first tile column / row leave the maximum of their rows of A / columns of B in a slot of the workspace, everybody
//     reads all slots (as in amax_cast_kernel: the value is its own flag, bit 31; nothing else is exchanged).  Nobody has to be resident for anybody
//     else to finish: those that have waited kScaledPatience see to the missing maxima together (missing_maxima);
//   - the factors known, the registers are rounded to FP8, into LDS where the fragments are read; of every row and column the
//     workgroups that share it write one chunk of 128 to the FP8 outputs in turn;
//   - products and sums are those of gemm_small_kernel in tiles of 32 x 32 (chunk c of 128 belongs to wave c % 8, the waves' sums are added in wave
//     order), so every result is bit for bit that of the separate launches.
// An operand is read and rounded once per tile that needs it (out of the caches), which bounds the sizes: see scaled_gemm_small_takes.
// 256 x 256 x 256 of fp32 8.9 -> 7.2 us (as a graph node 8.3 -> 7.1), 19 x 2048 x 256 10.8 -> 7.2, 64 x 960 x 194 10.8 -> 7.1, 32 x 6336 x 448
// 15.8 -> 11.3.  What is left is latency: the launch, one load, the exchange (a store and a load through memory), the end of the tile.
//
// This file is compiled once per pair of storage orders: -DFP8MM_LAYOUT.
#include "cast_common.hpp"
#include "gemm_small_tile.hpp"

#include <atomic>

namespace fp8mm {
namespace {

constexpr int kWaves = 8, kTileThreads = 64 * kWaves;
// 50 us: beside a product whose tiles hold the compute units for 240 us, 256 x 256 x 256 took 106 us a call with 50 or 200 us of patience, 150 - 175 with 10 or less
// (the units that a workgroup gives back go to the other product).
constexpr unsigned kScaledPatience = 5000;
static_assert((kCastSlots + 256) * sizeof(unsigned) <= FP8_AMAX_WORKSPACE_BYTES, "a slot per tile row or column");

// The vector without its first k elements (0 <= k < per_vec), zeros behind the rest.
template <int DT>
__device__ __forceinline__ u32x4 without_first(u32x4 v, int k)
{
    const int words = DT == FP8_F32 ? k : k >> 1;
    if (words & 2) v = (u32x4){v.z, v.w, 0u, 0u};
    if (words & 1) v = (u32x4){v.y, v.z, v.w, 0u};
    if (DT == FP8_BF16 && (k & 1))
        v = (u32x4){(v.x >> 16) | (v.y << 16), (v.y >> 16) | (v.z << 16), (v.z >> 16) | (v.w << 16), v.w >> 16};
    return v;
}

// The 32 rows of op(A) / columns of op(B) from t0 on, in their wide type: vector j of a thread holds per_vec elements at K index
// k0 + j STEP of a row (KC: element (r, k) at x[r K + k]) or columns at one K index (MC: at x[k ext + r]).  NV: vectors per thread.  RAGGED: the rows in
// memory (of K or ext elements, per_vec at least) end inside a vector: that one is loaded from the row's last elements and shifted.
template <int DT, bool KC, int NV, bool RAGGED>
struct Panel {
    typedef Operand<KC, 1, 2> Slab;                       // chunks of 128 along K
    static constexpr int PV = Elem<DT>::per_vec, ESZ = Elem<DT>::size;
    static constexpr int LANES = KC ? 16 : 32 / PV;       // that share a row
    static constexpr int STEP = KC ? 16 * PV : kTileThreads / LANES;      // K from one vector of a thread to the next: 128 (bf16) or 64
    static_assert(STEP == (DT == FP8_BF16 ? 128 : 64) && kTileThreads / 16 == 32, "the thread's vectors");
    const char* x;
    int64_t first, pitch, safe;                           // element of vector 0; elements between two vectors; a vector near by that is there
    int k0, K, to;                                        // K index of vector 0; K; where it goes in the first slab
    int over;                                             // MC: elements of the thread's vectors beyond the end of the row
    bool row;                                             // the thread's row / columns exist

    __device__ __forceinline__ void setup(const void* x_, int64_t ext, int K_, int64_t t0, int tid)
    {
        x = (const char*)x_;
        K = K_;
        const int r = tid / LANES, e = (tid % LANES) * PV;
        to = r * Slab::PITCH + e;
        if (KC) {
            row = t0 + r < ext;
            k0 = e;
            over = 0;
            first = (t0 + r) * K + e;
            pitch = STEP;
            safe = (t0 + (row ? r : 0)) * K;
        } else {
            row = t0 + e < ext;
            k0 = r;
            over = RAGGED && row && t0 + e + PV > ext ? (int)(t0 + e + PV - ext) : 0;
            first = (int64_t)r * ext + t0 + e;
            pitch = STEP * ext;
            safe = RAGGED ? 0 : t0 + (row ? e : 0);
        }
    }
    __device__ __forceinline__ bool here(int j) const { return row && k0 + j * STEP < K; }
    // how many elements of vector j, which is here, lie beyond the end of its row
    __device__ __forceinline__ int beyond(int j) const
    {
        if (!RAGGED) return 0;
        if (!KC) return over;
        const int b = k0 + j * STEP + PV - K;
        return b > 0 ? b : 0;
    }
    // Every vector is loaded, one near by in the place of one that is not there (with a choice whether to load, the compiler kept the registers
    // in scratch memory).
    __device__ __forceinline__ unsigned load(u32x4 (&v)[NV]) const
    {
        unsigned run = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] = *(const u32x4_any*)(x + (here(j) ? first + j * pitch - beyond(j) : safe) * ESZ);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const unsigned mask = here(j) ? ~0u : 0u;
            if (RAGGED) v[j] = without_first<DT>(v[j], here(j) ? beyond(j) : 0);
            v[j] = (u32x4){v[j].x & mask, v[j].y & mask, v[j].z & mask, v[j].w & mask};
            run = vec_mag_max<DT>(v[j], run);
        }
        return run_to_bits<DT>(run);
    }
    // Rounded, into the slabs (zeros behind the end of K), and to q where the chunk is this workgroup's of the `sharers` that have it.
    template <int FMT>
    __device__ __forceinline__ void cast(const u32x4 (&v)[NV], float s, uint8_t* slabs, uint8_t* __restrict__ q, unsigned sharer, unsigned sharers) const
    {
        constexpr int VPI = DT == FP8_BF16 ? 2 : 4, PER_CHUNK = 128 / STEP;
        const int vecs = (K + 127) / 128 * PER_CHUNK;
        unsigned turn = sharer;                           // chunks from here to the next one of this workgroup's
#pragma unroll
        for (int g = 0; g < NV / VPI; ++g) {
            if (g > 0 && g * VPI >= vecs) continue;
            u32x4 item[VPI];
            float y[16];
#pragma unroll
            for (int i = 0; i < VPI; ++i) item[i] = v[g * VPI + i];
            scale_item<DT>(item, s, y);
            const u32x4 o = encode16<FMT, kCastCvt>(y);
#pragma unroll
            for (int i = 0; i < VPI; ++i) {
                const int j = g * VPI + i, c = j / PER_CHUNK;
                if (j < vecs) {
                    const auto piece = Piece<DT>::of(o, i);
                    uint8_t* at = slabs + c * Slab::SLAB + to + (KC ? (j % PER_CHUNK) * STEP : (j % PER_CHUNK) * STEP * Slab::PITCH);
                    if constexpr (DT == FP8_BF16) *LDS_PTR(u32x2, at) = piece; else *LDS_PTR(unsigned, at) = piece;
                    if (turn == 0 && here(j)) {
                        uint8_t* out = q + first + j * pitch;
                        if (!RAGGED || beyond(j) == 0) *(typename Piece<DT>::type*)out = piece;
                        else for (int n = 0; n < PV - beyond(j); ++n) out[n] = (uint8_t)(o[(PV / 4) * i + (n >> 2)] >> (8 * (n & 3)));
                    }
                }
                if (j % PER_CHUNK == PER_CHUNK - 1) turn = turn == 0 ? sharers - 1 : turn - 1;
            }
        }
    }
};

// The largest magnitude of the 32 rows of op(A) / columns of op(B) from t0 on, by the workgroup; valid in thread 0.  (Small loops of their own: with
// Panel's loads in their place the compiler kept addresses for these all through the kernel, and 256 x 256 x 256 took 0.2 us longer.)
template <int DT, bool KC>
__device__ __forceinline__ unsigned panel_max(const void* x, int64_t ext, int K, int64_t t0)
{
    constexpr int PV = Elem<DT>::per_vec, ESZ = Elem<DT>::size;
    const int rows = ext - t0 < 32 ? (int)(ext - t0) : 32;
    unsigned run = 0, r = 0;
    if (KC) {                                             // one run of elements
        const char* first = (const char*)x + t0 * K * ESZ;
        const int n = rows * K, tail = n / PV * PV + threadIdx.x;
#pragma unroll 1
        for (int i = threadIdx.x; i < n / PV; i += kTileThreads) run = vec_mag_max<DT>(((const u32x4_any*)first)[i], run);
        if (tail < n) r = scalar_mag<DT>(first, tail);
    } else {                                              // a K index per thread
#pragma unroll 1
        for (int k = threadIdx.x; k < K; k += kTileThreads) {
            const char* first = (const char*)x + (k * ext + t0) * ESZ;
            int c = 0;
#pragma unroll 1
            for (; c + PV <= rows; c += PV) run = vec_mag_max<DT>(*(const u32x4_any*)(first + c * ESZ), run);
#pragma unroll 1
            for (; c < rows; ++c) r = max(r, scalar_mag<DT>(first, c));
        }
    }
    return block_max_u32<kTileThreads>(max(r, run_to_bits<DT>(run)));
}

struct ScaledArgs {
    const void *a, *b;
    uint8_t *qa, *qb;
    float *amax, *scale;
    unsigned* ws;
    unsigned patience;
};

template <int DT, int FMT_A, int FMT_B, int ACC, bool A_KC, bool B_KC, int NV, bool RAGGED>
__global__ __launch_bounds__(kTileThreads) void scaled_gemm_small_kernel(ScaledArgs p, void* __restrict__ C, int M, int N, int K, int out_kind)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    typedef Operand<A_KC, 1, 2> OpA;
    typedef Operand<B_KC, 1, 2> OpB;
    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // tiles as in gemm_small_kernel: down the rows of C, a contiguous run per XCD
    const unsigned tiles_m = (M + 31) / 32, tiles_n = (N + 31) / 32, total = gridDim.x;
    const unsigned xcd = blockIdx.x % 8, share = total / 8, rem = total % 8;
    const unsigned t = xcd * share + (xcd < rem ? xcd : rem) + blockIdx.x / 8;
    const unsigned tm = t % tiles_m, tn = t / tiles_m;
    const int64_t m0 = tm * 32, n0 = tn * 32;
    unsigned* ws_a = p.ws;
    unsigned* ws_b = p.ws + FP8_AMAX_WORKSPACE_BYTES / 4;

    Panel<DT, A_KC, NV, RAGGED> a; Panel<DT, B_KC, NV, RAGGED> b;
    a.setup(p.a, M, K, m0, tid);
    b.setup(p.b, N, K, n0, tid);
    u32x4 va[NV], vb[NV];
    const unsigned run_a = a.load(va), run_b = b.load(vb);

    __shared__ unsigned part_a[kWaves], part_b[kWaves], largest[2];
    __shared__ unsigned long long absent[5];                 // panels whose maximum has not come, those of B behind those of A
    __shared__ bool complete;                                // there are none
    unsigned ticket = 0;                                     // of the workgroup among those that have read all slots (first lane)
    {
        const unsigned ma = wave_max_u32(run_a), mb = wave_max_u32(run_b);
        if (l == 0) { part_a[w] = ma; part_b[w] = mb; }
        __syncthreads();
    }
    if (w == 0) {
        // lanes 0 .. 7 have the waves' maxima
        const unsigned own_a = wave_max_u32(l < kWaves ? part_a[l] : 0u), own_b = wave_max_u32(l < kWaves ? part_b[l] : 0u);
        if (l == 0 && tn == 0) __hip_atomic_store(&ws_a[kCastSlots + tm], own_a | 0x80000000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (l == 0 && tm == 0) __hip_atomic_store(&ws_b[kCastSlots + tn], own_b | 0x80000000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long began = wall_clock64();
        unsigned ma = own_a, mb = own_b;
        bool here = true;
        auto collect = [&](const unsigned* slots, unsigned count, unsigned& m) {
            for (unsigned i = l; i < count; i += 64) {
                unsigned v = 0;
                while (!(v >> 31)) {
                    v = __hip_atomic_load(&slots[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (wall_clock64() - began > p.patience) break;
                }
                here = here && v >> 31;
                m = max(m, v & 0x7fffffffu);
            }
        };
        collect(ws_a + kCastSlots, tiles_m, ma);
        collect(ws_b + kCastSlots, tiles_n, mb);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0x0070);                  // vmcnt(0): the own maxima have been acknowledged
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        const bool everybody = __all(here);
        ma = wave_max_u32(ma); mb = wave_max_u32(mb);
        if (l == 0) {
            largest[0] = ma; largest[1] = mb;
            complete = everybody;
            // (nobody waits for the answer before the end: waited for here it was 0.8 us of every workgroup's time)
            if (everybody) ticket = __hip_atomic_fetch_add(&ws_a[kCastDone], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (__builtin_expect(!complete, 0)) {                                     // (never, unless other work held compute units for as long)
        const unsigned panels = tiles_m + tiles_n;
        if (tid == 0)
            for (unsigned k = 0; 64 * k < panels; ++k) absent[k] = panels - 64 * k >= 64 ? ~0ull : (1ull << (panels - 64 * k)) - 1;
        __syncthreads();
        missing_maxima(absent, panels, t, [&](unsigned i) { return p.ws + kCastSlots + (i < tiles_m ? i : FP8_AMAX_WORKSPACE_BYTES / 4 + i - tiles_m); },
                       [&](unsigned i) { return i < tiles_m ? panel_max<DT, A_KC>(p.a, M, K, i * 32) : panel_max<DT, B_KC>(p.b, N, K, (i - tiles_m) * 32); },
                       [&](unsigned i, unsigned m) { atomicMax(&largest[i < tiles_m ? 0 : 1], m); });
        if (tid == 0) {
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0): the maxima of others have been acknowledged
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            ticket = __hip_atomic_fetch_add(&ws_a[kCastDone], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    const float amax_a = as_f32(largest[0]), amax_b = as_f32(largest[1]);
    const float sa = scale_rule(amax_a, FMT_A), sb = scale_rule(amax_b, FMT_B);
    if (t == 0 && tid == 0) { p.amax[0] = amax_a; p.amax[1] = amax_b; p.scale[0] = sa; p.scale[1] = sb; }

    const int chunks = (K + 127) / 128;
    uint8_t* slabs_b = lds + chunks * OpA::SLAB;
    // chunk c of a row block is written by the workgroup of tile column c mod tiles_n (the same with columns and tile rows)
    a.template cast<FMT_A>(va, sa, lds, p.qa, tn, tiles_n);
    b.template cast<FMT_B>(vb, sb, slabs_b, p.qb, tm, tiles_m);
    __syncthreads();

    v16f acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    const OpA oa{}; const OpB ob{};
    for (int c = w; c < chunks; c += kWaves) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            v8i fa[1], fb[1];
            oa.fragments(lds + c * OpA::SLAB, sub, l, fa);
            ob.fragments(slabs_b + c * OpB::SLAB, sub, l, fb);
            if (ACC == ACC_FP8) {
                acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[0], fa[0], acc, FMT_B, FMT_A, 0, 0, 0, 0);
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(widen8<FMT_B>(fb[0][2 * s], fb[0][2 * s + 1]), widen8<FMT_A>(fa[0][2 * s], fa[0][2 * s + 1]),
                                                                      acc, 0, 0, 0);
            }
        }
    }

    // the waves' sums meet in LDS and are added in wave order; a thread has 4 consecutive columns of a row (as in gemm_small_kernel)
    constexpr int RED = 32 * RED_PITCH;                   // floats of a wave's sums
    const float r = (float)(1.0 / ((double)sa * (double)sb));
    __syncthreads();                                      // the slabs are done with
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *LDS_PTR(v4f, (float*)lds + w * RED + (l & 31) * RED_PITCH + 8 * q + 4 * (l >> 5)) =
            (v4f){acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    __syncthreads();
    const int64_t gm = m0 + (tid >> 3), gn = n0 + 4 * (tid & 7);
    if (tid < 32 * 8 && gm < M && gn < N) {
        const float* red = (const float*)lds + (tid >> 3) * RED_PITCH + 4 * (tid & 7);
        v4f sum = *LDS_PTR(v4f, red);
#pragma unroll
        for (int v = 1; v < kWaves; ++v) sum += *LDS_PTR(v4f, red + v * RED);
        sum *= r;
        const int left = N - gn < 4 ? (int)(N - gn) : 4;
        if (out_kind == OUT_F32) {
            float* out = (float*)C + gm * N + gn;
            if (left == 4 && ((uintptr_t)out & 15) == 0) *(v4f*)out = sum;
            else for (int e = 0; e < left; ++e) out[e] = e == 0 ? sum.x : e == 1 ? sum.y : e == 2 ? sum.z : sum.w;
        } else {
            unsigned short* out = (unsigned short*)C + gm * N + gn;
            const unsigned lo = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){sum.x, sum.y}, v2bf));
            const unsigned hi = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){sum.z, sum.w}, v2bf));
            if (left == 4 && ((uintptr_t)out & 7) == 0) *(v2i*)out = (v2i){(int)lo, (int)hi};
            else for (int e = 0; e < left; ++e) out[e] = (unsigned short)((e < 2 ? lo : hi) >> (16 * (e & 1)));
        }
    }
    if (w == 0 && (unsigned)__builtin_amdgcn_readfirstlane((int)ticket) == total - 1) {
        for (unsigned i = l; i < tiles_m; i += 64) __hip_atomic_store(&ws_a[kCastSlots + i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (unsigned i = l; i < tiles_n; i += 64) __hip_atomic_store(&ws_b[kCastSlots + i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (l == 0) __hip_atomic_store(&ws_a[kCastDone], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int DT, int FA, int FB, int ACC, bool A_KC, bool B_KC, int NV, bool RAGGED>
int launch_typed(const GemmArgs& g, const ScaledArgs& p)
{
    auto kern = scaled_gemm_small_kernel<DT, FA, FB, ACC, A_KC, B_KC, NV, RAGGED>;
    const int lds = scaled_gemm_small_lds(g);
    if (lds > 65536) {
        // more dynamic LDS than the default limit: raised once per device
        static std::atomic<unsigned long long> attr_set{0ull};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return fail(FP8_ERR_DEVICE, "hipGetDevice failed");
        const unsigned long long bit = 1ull << (dev & 63);
        if (dev >= 64 || !(attr_set.load(std::memory_order_relaxed) & bit)) {
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kScaledSmallLds);
            if (e != hipSuccess) return fail(FP8_ERR_DEVICE, "hipFuncSetAttribute(LDS=%d): %s", kScaledSmallLds, hipGetErrorString(e));
            if (dev < 64) attr_set.fetch_or(bit, std::memory_order_relaxed);
        }
    }
    const int64_t tiles = ((g.M + 31) / 32) * ((g.N + 31) / 32);
    enqueue(kern, dim3((unsigned)tiles), dim3(kTileThreads), lds, g.stream, p, g.C, (int)g.M, (int)g.N, (int)g.K, g.ep.out_kind);
    return check_launch("scaled gemm (one launch)");
}

template <int DT, int FA, int FB, int ACC, bool RAGGED>
int launch_vecs(const GemmArgs& g, const ScaledArgs& p)
{
    constexpr bool A_KC = (FP8MM_LAYOUT & 2) == 0, B_KC = (FP8MM_LAYOUT & 1) != 0;
    constexpr int MOST = kScaledSmallRow / 256;          // vectors per thread for the longest K
    // (with eight vectors a thread, of which these rows have five or six, 295 x 332 x 576 lost as a graph node: 9.8 us apart, 10.1 together, now 9.7)
    if constexpr (!RAGGED && DT == FP8_BF16)
        if (g.K * Elem<DT>::size > kScaledSmallRow / 2 && g.K * Elem<DT>::size <= kScaledSmallRow / 4 * 3)
            return launch_typed<DT, FA, FB, ACC, A_KC, B_KC, MOST / 4 * 3, false>(g, p);
    if constexpr (!RAGGED)
        if (g.K * Elem<DT>::size > kScaledSmallRow / 2) return launch_typed<DT, FA, FB, ACC, A_KC, B_KC, MOST, false>(g, p);
    return launch_typed<DT, FA, FB, ACC, A_KC, B_KC, MOST / 2, RAGGED>(g, p);   // (ragged rows: only so long, see scaled_gemm_small_takes)
}

template <int DT, int FA, int FB, int ACC>
int launch_rows(const GemmArgs& g, const ScaledArgs& p)
{
    constexpr int PV = Elem<DT>::per_vec;
    return (g.transA ? g.M : g.K) % PV || (g.transB ? g.K : g.N) % PV ? launch_vecs<DT, FA, FB, ACC, true>(g, p) : launch_vecs<DT, FA, FB, ACC, false>(g, p);
}

template <int DT, int FA, int FB>
int launch_acc(const GemmArgs& g, const ScaledArgs& p)
{
    return g.acc == ACC_FP8 ? launch_rows<DT, FA, FB, ACC_FP8>(g, p) : launch_rows<DT, FA, FB, ACC_F16>(g, p);
}

template <int DT>
int launch_formats(const GemmArgs& g, const ScaledArgs& p)
{
    if (g.fmtA == FP8_E4M3) return g.fmtB == FP8_E4M3 ? launch_acc<DT, FP8_E4M3, FP8_E4M3>(g, p) : launch_acc<DT, FP8_E4M3, FP8_E5M2>(g, p);
    return g.fmtB == FP8_E4M3 ? launch_acc<DT, FP8_E5M2, FP8_E4M3>(g, p) : launch_acc<DT, FP8_E5M2, FP8_E5M2>(g, p);
}

}  // namespace

#if !defined(FP8MM_LAYOUT)
#error "compile with -DFP8MM_LAYOUT=0..3 (2 * transA + transB)"
#endif

int FP8MM_SCALED_NAME(FP8MM_LAYOUT)(const GemmArgs& g, const void* a, const void* b, int in_dtype, float* amax_out, float* scale_out, void* workspace)
{
    const ScaledArgs p{a, b, (uint8_t*)g.A, (uint8_t*)g.B, amax_out, scale_out, (unsigned*)workspace, patience(kScaledPatience)};
    return in_dtype == FP8_F32 ? launch_formats<FP8_F32>(g, p) : launch_formats<FP8_BF16>(g, p);
}

}  // namespace fp8mm
