// Pieces shared by the translation units of the amax / cast kernels (gfx950).
#pragma once

#include "common.hpp"
#include "fp8_decode.hpp"
#include "fp8_encode.hpp"

namespace fp8mm {
namespace {

constexpr int kThreads = 256;
constexpr int kAmaxBlocks = 256 * 4;      // read-only stream: 32 KB chunks dealt to this many workgroups measured best
// read+write stream: short contiguous runs of 16 384 elements per workgroup measured best at every
// size (6.04 10^8 bf16 elements: 290 us, against 320 us when the grid stopped growing at 16 384
// workgroups); the limit only keeps the grid dimension in range
constexpr int kCastBlocks = 1 << 20;
constexpr int kMultiMax = FP8_MULTI_MAX;  // tensors per launch of the multi-tensor forms
constexpr size_t kStreamingStoreBytes = (size_t)384 << 20;   // outputs from this size on are stored non-temporally

// Words of the amax workspace (4096 a tensor): tickets and partial maxima of the one-launch amax (amax_finish_ticket), then those of
// the launches in which the maxima of a tensor's parts meet in slots (amax_cast_kernel, scaled_gemm_small_kernel).
constexpr unsigned kTicketGroup = 32;
constexpr unsigned kTicketPartials = 32 * (1 + kAmaxBlocks / kTicketGroup);
constexpr unsigned kCastDone = kTicketPartials + kAmaxBlocks;        // workgroups that have read all slots
constexpr unsigned kCastSlots = kCastDone + 32;                      // ... and the slots (nothing else uses these words)

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// Vectors at any address: the target's global loads and stores take them as one instruction.
typedef u32x4 u32x4_any __attribute__((aligned(1)));
typedef u32x2 u32x2_any __attribute__((aligned(1)));
typedef unsigned u32_any __attribute__((aligned(1)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------------------------------
// amax.  Magnitude bits of IEEE numbers order like unsigned integers (Section 3.1 relies on
// the same property for FP8), NaN patterns sort above infinity, so an unsigned max of the
// sign-stripped bits is the NaN-propagating amax.  bfloat16 pairs are reduced as packed
// 16-bit integers.
// ------------------------------------------------------------------------------------------
template <int DT> struct Elem;
template <> struct Elem<FP8_F32>  { static constexpr int size = 4; static constexpr int per_vec = 4; };
template <> struct Elem<FP8_BF16> { static constexpr int size = 2; static constexpr int per_vec = 8; };

template <int DT>
__device__ __forceinline__ unsigned vec_mag_max(u32x4 v, unsigned run)
{
    if (DT == FP8_F32) {
        unsigned m0 = v.x & 0x7fffffffu, m1 = v.y & 0x7fffffffu;
        unsigned m2 = v.z & 0x7fffffffu, m3 = v.w & 0x7fffffffu;
        m0 = m0 > m1 ? m0 : m1;
        m2 = m2 > m3 ? m2 : m3;
        m0 = m0 > m2 ? m0 : m2;
        return run > m0 ? run : m0;
    } else {
        u16x2 r = __builtin_bit_cast(u16x2, run);
        r = __builtin_elementwise_max(r, __builtin_bit_cast(u16x2, v.x & 0x7fff7fffu));
        r = __builtin_elementwise_max(r, __builtin_bit_cast(u16x2, v.y & 0x7fff7fffu));
        r = __builtin_elementwise_max(r, __builtin_bit_cast(u16x2, v.z & 0x7fff7fffu));
        r = __builtin_elementwise_max(r, __builtin_bit_cast(u16x2, v.w & 0x7fff7fffu));
        return __builtin_bit_cast(unsigned, r);
    }
}

// Magnitude bits of one element, as the bits of an fp32 number.
template <int DT>
__device__ __forceinline__ unsigned scalar_mag(const void* x, size_t i)
{
    if (DT == FP8_F32) return ((const unsigned*)x)[i] & 0x7fffffffu;
    return ((unsigned)(((const unsigned short*)x)[i] & 0x7fffu)) << 16;
}

// Packed running maximum (see vec_mag_max) -> sign-stripped fp32 bits.
template <int DT>
__device__ __forceinline__ unsigned run_to_bits(unsigned run)
{
    if (DT == FP8_F32) return run;
    const u16x2 p = __builtin_bit_cast(u16x2, run);
    return (unsigned)(p.x > p.y ? p.x : p.y) << 16;
}

// Largest value over the lanes of each row of 16, in its first lane / over all 64 lanes, in every lane; all lanes active.
// Lanes exchange within the vector registers (a shuffle goes through the LDS unit and takes about a hundred clocks
// a step: the six steps were a quarter of a microsecond of every small kernel).
__device__ __forceinline__ unsigned row_max_u32(unsigned v)
{
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x101, 0xf, 0xf, false));      // row_shl:1, 2, 4, 8
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x102, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x104, 0xf, 0xf, false));
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x108, 0xf, 0xf, false));
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned v)
{
    v = row_max_u32(v);
    const unsigned a = (unsigned)__builtin_amdgcn_readlane((int)v, 0), b = (unsigned)__builtin_amdgcn_readlane((int)v, 16);
    const unsigned c = (unsigned)__builtin_amdgcn_readlane((int)v, 32), d = (unsigned)__builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}

template <int THREADS = kThreads>
__device__ __forceinline__ unsigned block_max_u32(unsigned v)
{
    __shared__ unsigned part[THREADS / 64];
    v = wave_max_u32(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) v = v > part[w] ? v : part[w];
    }
    return v;   // valid in thread 0
}

// How long a workgroup waits for the slots: `ticks` of the 100 MHz clock, or not at all.
inline unsigned patience(unsigned ticks) { return knob(FP8_KNOB_PATIENCE) ? 0u : ticks; }

// For a workgroup that has waited long enough: the maxima of the parts whose slots were still empty.  absent: a bit in LDS for each of the
// `count` parts, set where the maximum has not come.  The workgroups that get here share what is missing, so that together they read each part
// about once: each starts at another part (`turn` is its number), leaves what it finds in that part's slot (the value is the same whoever finds it)
// and looks at the slots again before the next.  At most `count` rounds.  slot(i): where the maximum of part i goes; part_max(i): the workgroup takes
// it from the tensor (a barrier inside; valid in thread 0); take(i, m): the maximum of part i is m.  All threads call it.  The caller waits for the
// stores of thread 0 before it counts the workgroup among the readers, or they could land behind the clearing of the slots.
// (Each workgroup on its own took all missing parts: four streams of 2048 x 4096 x 2048 steps in bf16 took 2064 us a call, now 178; in
// separate launches 160 - 180.)
template <typename Slot, typename PartMax, typename Take>
__device__ __forceinline__ void missing_maxima(unsigned long long* absent, unsigned count, unsigned turn, Slot slot, PartMax part_max, Take take)
{
    for (;;) {
        if (threadIdx.x < 64) {
            for (unsigned k = 0; 64 * k < count; ++k) {
                const unsigned i = 64 * k + threadIdx.x;
                bool missing = absent[k] >> threadIdx.x & 1;
                if (missing) {
                    const unsigned p = __hip_atomic_load(slot(i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (p >> 31) { take(i, p & 0x7fffffffu); missing = false; }
                }
                const unsigned long long left = __ballot(missing);
                if (threadIdx.x == 0) absent[k] = left;
            }
        }
        __syncthreads();
        unsigned left = 0;
        for (unsigned k = 0; 64 * k < count; ++k) left += (unsigned)__popcll(absent[k]);
        if (left == 0) return;
        unsigned skip = turn % left, k = 0;               // the part: this many missing ones from the first
        while (skip >= (unsigned)__popcll(absent[k])) skip -= (unsigned)__popcll(absent[k++]);
        unsigned long long bits = absent[k];
        for (; skip > 0; --skip) bits &= bits - 1;
        const unsigned i = 64 * k + (unsigned)__builtin_ctzll(bits);
        const unsigned m = part_max(i);
        if (threadIdx.x == 0) {
            __hip_atomic_store(slot(i), m | 0x80000000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            take(i, m);
            absent[k] &= ~(1ull << (i & 63));
        }
        __syncthreads();
    }
}

__global__ void store_u32_kernel(unsigned* p, unsigned v) { *p = v; }

// ------------------------------------------------------------------------------------------
// scale = fmt_max / amax, one IEEE single division (Section 2; Table 1 "Max normal";
// Section 3.2: any real value).  Degenerate amax (0, NaN, inf) or a quotient that is not
// finite gives 1.
// ------------------------------------------------------------------------------------------
__host__ __device__ inline float scale_rule(float amax, int fmt)
{
    const float fmax = fmt == FP8_E4M3 ? 448.0f : 57344.0f;
    if (!(amax > 0.0f) || amax > 3.4028234663852886e38f) return 1.0f;
    const float s = fmax / amax;
    if (!(s <= 3.4028234663852886e38f)) return 1.0f;
    return s;
}

template <int DT>
__device__ __forceinline__ float load_scalar(const void* x, size_t i)
{
    if (DT == FP8_F32) return ((const float*)x)[i];
    return as_f32((unsigned)((const unsigned short*)x)[i] << 16);
}

// The 16 elements of one work item, scaled: from 2 (bf16) or 4 (fp32) 16-byte vectors.
template <int DT>
__device__ __forceinline__ void scale_item(const u32x4 (&v)[DT == FP8_BF16 ? 2 : 4], float s, float (&y)[16])
{
    if (DT == FP8_BF16) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                y[8 * j + 2 * d] = as_f32(v[j][d] << 16) * s;
                y[8 * j + 2 * d + 1] = as_f32(v[j][d] & 0xffff0000u) * s;
            }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int d = 0; d < 4; ++d) y[4 * j + d] = as_f32(v[j][d]) * s;
    }
}

// How the vector kernels deal the work to lanes.  A lane that took 16 consecutive elements (32 or 64
// bytes of input) itself would make every load instruction of its wave touch 64 lines for a half
// or a quarter of their bytes.  Instead a lane takes single 16-byte vectors, kThreads vectors apart
// (every load instruction of a wave then reads 1 KB of consecutive bytes), rounds 16 elements from
// 2 (bf16) or 4 (fp32) such vectors at a time with the common routine, and stores the output bytes
// of each vector as one piece of 8 (bf16) or 4 (fp32) bytes, again consecutive across the wave.
// Measured on 2^28 elements against 16 consecutive elements per lane: bf16 6.4 -> 6.7 TB/s,
// fp32 4.25 -> 6.2 TB/s.
template <int DT> struct Piece;
template <> struct Piece<FP8_BF16> {
    typedef u32x2_any type;
    static __device__ __forceinline__ type of(const u32x4& o, int k) { return (u32x2){o[2 * k], o[2 * k + 1]}; }
};
template <> struct Piece<FP8_F32> {
    typedef u32_any type;
    static __device__ __forceinline__ type of(const u32x4& o, int k) { return o[k]; }
};

// One group: the loaded vectors in[k] = xv[v + k * THREADS], k < VPI -> the pieces
// qp[v + k * THREADS]; only the first `count` pieces are stored.  AMAX: the running packed maximum of the
// vectors is kept in `run` (vectors beyond `count` must be zeros).
template <int DT, int FMT, int PATH, bool NTS, bool AMAX, int THREADS = kThreads>
__device__ __forceinline__ void cast_group(const u32x4* in, typename Piece<DT>::type* __restrict__ qp,
                                           size_t v, int count, float s, unsigned& run)
{
    constexpr int VPI = DT == FP8_BF16 ? 2 : 4;
    u32x4 item[VPI];
#pragma unroll
    for (int k = 0; k < VPI; ++k) {
        item[k] = in[k];
        if (AMAX) run = vec_mag_max<DT>(item[k], run);
    }
    float y[16];
    scale_item<DT>(item, s, y);
    const u32x4 o = encode16<FMT, PATH>(y);
#pragma unroll
    for (int k = 0; k < VPI; ++k) {
        if (k < count) {
            typename Piece<DT>::type* dst = &qp[v + (size_t)k * THREADS];
            if (NTS) __builtin_nontemporal_store(Piece<DT>::of(o, k), dst); else *dst = Piece<DT>::of(o, k);
        }
    }
}

// A lane's walk over the vectors [vlo, vhi) of its workgroup: 8 vectors per step, all loads of a
// step issued before the first conversion; then the remainder, group by group.
template <int DT, int FMT, int PATH, bool NTS, bool AMAX, int THREADS = kThreads>
__device__ __forceinline__ void cast_run(const u32x4_any* __restrict__ xv, typename Piece<DT>::type* __restrict__ qp,
                                         size_t vlo, size_t vhi, float s, unsigned& run)
{
    constexpr int VPI = DT == FP8_BF16 ? 2 : 4;
    size_t v = vlo + threadIdx.x;
    for (; v + 7 * THREADS < vhi; v += 8 * THREADS) {
        u32x4 in[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) in[k] = __builtin_nontemporal_load(&xv[v + (size_t)k * THREADS]);
#pragma unroll
        for (int g = 0; g < 8 / VPI; ++g)
            cast_group<DT, FMT, PATH, NTS, AMAX, THREADS>(in + g * VPI, qp, v + (size_t)g * VPI * THREADS, VPI, s, run);
    }
    for (; v < vhi; v += VPI * THREADS) {
        const size_t left = (vhi - v + THREADS - 1) / THREADS;        // vectors of this lane still there
        const int count = left < (size_t)VPI ? (int)left : VPI;
        u32x4 in[VPI];
#pragma unroll
        for (int k = 0; k < VPI; ++k)
            in[k] = k < count ? __builtin_nontemporal_load(&xv[v + (size_t)k * THREADS]) : (u32x4){0u, 0u, 0u, 0u};
        cast_group<DT, FMT, PATH, NTS, AMAX, THREADS>(in, qp, v, count, s, run);
    }
}

inline int grid_for(size_t work_items, int max_blocks)
{
    size_t b = (work_items + kThreads - 1) / kThreads;
    if (b < 1) b = 1;
    if (b > (size_t)max_blocks) b = max_blocks;
    return (int)b;
}


}  // namespace
}  // namespace fp8mm
