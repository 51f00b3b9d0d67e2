// amax reduction, scale computation and the FP8 cast for gfx950 (MI355X).
//
// All three are HBM-streaming kernels: every lane moves 16-byte vectors, the arithmetic per
// element is a handful of VALU instructions.  The paper's scheme (arXiv 2209.05433,
// Section 2) is: find the largest magnitude of the tensor, pick scale = fmt_max / amax,
// multiply every element by the scale and round it to E4M3 / E5M2 (Table 1) with
// saturation.
#include "common.hpp"
#include "fp8_decode.hpp"
#include "fp8_encode.hpp"
#include "cast_common.hpp"

#include <algorithm>

namespace fp8mm {
namespace {

// nvec whole vectors, at any address, then n - nvec*per_vec tail elements.  Every workgroup takes
// chunks of 32 KB (8 vectors per lane, all loaded before the first compare).  In the one-launch form there are up to four workgroups per
// compute unit; with an atomic on one cell, one: they end together, and the more there are the longer they queue (24 MB of bf16 256 /
// 512 / 1024 workgroups 8.1 / 9.3 / 12.4 us, 32 MB 9.1 / 11.0 / 22.0, 128 MB 22.1 / 22.4 / 30.4, 600 MB 86.7 / 89.0 / 88.2).
// The one-launch form cuts tensors of less than 1 MB into
// chunks of 8 KB: their time is the latency of a few loads (64 KB of bf16 4.1 -> 3.8 us; 4 MB of fp32 5.1 -> 5.5 and
// 10 MB of bf16 5.8 -> 6.6, all in chunks of 8 KB); up to 64 KB one workgroup reads the tensor alone, 16 vectors per lane in
// flight: no tickets are drawn, each of which is a round trip to memory.  The line lies where amax and the cast that follows
// it, together, gain on a tensor that another kernel has just written: one workgroup fetches what lies in eight L2s, and the cast's
// workgroups again what lies in its own (amax + cast in chunks of 8 KB / by one workgroup: 16 KB of bf16 5.1 / 4.5 us, 32 KB 5.5 / 4.75,
// 64 KB 5.7 / 5.5, but 96 KB 5.7 / 6.45, 128 KB 5.8 / 6.6; of fp32 64 KB 6.05 / 5.4, 96 KB 6.2 / 6.7).
constexpr int kAmaxVecs = 8;                                         // per lane and chunk
constexpr int kAmaxVecsSmall = 2;
constexpr size_t kAmaxSmallBelow = (size_t)32 * kThreads * kAmaxVecs;    // vectors
constexpr size_t kAmaxAtomics = 256;                                 // workgroups that share a cell
constexpr int kAmaxVecsAlone = 16;
constexpr size_t kAmaxAloneBelow = (size_t)kThreads * kAmaxVecsAlone;      // vectors that one workgroup reads alone: 64 KB

// Last step of the amax kernels in their one-launch form (fp8_amax_scale): no cell has to be
// cleared beforehand and the scale comes out of the same launch.  Every workgroup leaves its
// maximum in the workspace and takes a ticket; the workgroup that draws the last ticket reduces the
// gridDim.x partial maxima, writes amax and scale = fmt_max / amax.  Tickets are drawn in two levels
// (groups of kTicketGroup workgroups, then one ticket per group): a thousand workgroups that finish
// together and draw from one counter queue up at that counter for longer than small tensors take
// to read.  Every counter is put back to 0 by the workgroup that drew its last ticket.
// Workspace words: [0] top counter; [32 (1 + g)] counter of group g (one 128-byte line each);
// [kTicketPartials + b] partial maximum of workgroup b.
// Ordering: the partial maximum is stored with an agent-scope atomic store (written through to where
// every other workgroup sees it) and has been acknowledged (vmcnt) before the ticket is drawn; the
// reader draws the last ticket before it loads, again with agent-scope atomic loads.  No other
// data is exchanged, so no cache-wide write-back or invalidate is needed.
// r: the workgroup's maximum, valid in thread 0.

__device__ __forceinline__ unsigned draw_ticket(unsigned* counter)
{
    return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// bid, grid: the workgroup's number and the number of workgroups that work on this tensor.
__device__ __forceinline__ void amax_finish_ticket(unsigned r, unsigned* __restrict__ ws, int fmt,
                                                   float* __restrict__ amax_out, float* __restrict__ scale_out,
                                                   unsigned bid, unsigned grid)
{
    if (grid == 1) {
        if (threadIdx.x == 0) {
            *amax_out = as_f32(r);
            if (scale_out) *scale_out = scale_rule(as_f32(r), fmt);
        }
        return;
    }
    __shared__ bool last;
    if (threadIdx.x == 0) {
        __hip_atomic_store(&ws[kTicketPartials + bid], r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);            // (the compiler keeps the three steps in this order)
        __builtin_amdgcn_s_waitcnt(0x0070);                 // vmcnt(0) (and lgkmcnt(0)): the store has been acknowledged
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        const unsigned g = bid / kTicketGroup, groups = (grid + kTicketGroup - 1) / kTicketGroup;
        const unsigned members = min(kTicketGroup, grid - g * kTicketGroup);
        bool l = false;
        if (draw_ticket(&ws[32 * (1 + g)]) == members - 1) {
            __hip_atomic_store(&ws[32 * (1 + g)], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            l = groups == 1 || draw_ticket(&ws[0]) == groups - 1;
        }
        last = l;
    }
    __syncthreads();
    if (!last) return;
    unsigned m = 0;
    for (unsigned i = threadIdx.x; i < grid; i += kThreads) {
        const unsigned p = __hip_atomic_load(&ws[kTicketPartials + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        m = m > p ? m : p;
    }
    m = block_max_u32(m);
    if (threadIdx.x == 0) {
        const float a = as_f32(m);
        *amax_out = a;
        if (scale_out) *scale_out = scale_rule(a, fmt);
        __hip_atomic_store(&ws[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The maximum over the chunks (of kThreads VECS vectors) that workgroup `bid` of `grid` takes, into run.
// The whole chunks first (a loop without tests: with the partial one in it the compiler shared loads
// between the two cases and waited for all of them, 83 -> 109 us on 2^28 elements); in the partial one
// the lanes beyond the end read the last vector again.
template <int DT, int VECS>
__device__ __forceinline__ void amax_chunks(const u32x4_any* xv, size_t nvec, unsigned bid, unsigned grid, unsigned (&run)[4])
{
    constexpr size_t CHUNK = (size_t)kThreads * VECS;
    const size_t whole = nvec / CHUNK;
    for (size_t c = bid; c < whole; c += grid) {
        const u32x4_any* p = xv + c * CHUNK + threadIdx.x;
        u32x4 v[VECS];
#pragma unroll
        for (int j = 0; j < VECS; ++j) v[j] = __builtin_nontemporal_load(p + j * kThreads);
#pragma unroll
        for (int j = 0; j < VECS; ++j) run[j & 3] = vec_mag_max<DT>(v[j], run[j & 3]);
    }
    if (whole * CHUNK < nvec && whole % grid == bid) {
        u32x4 v[VECS];
#pragma unroll
        for (int j = 0; j < VECS; ++j) {
            const size_t i = whole * CHUNK + threadIdx.x + j * kThreads;
            v[j] = xv[i < nvec ? i : nvec - 1];
        }
#pragma unroll
        for (int j = 0; j < VECS; ++j) run[j & 3] = vec_mag_max<DT>(v[j], run[j & 3]);
    }
}

// Workgroups for a tensor of nvec vectors.
inline unsigned amax_grid(size_t nvec, bool ticket)
{
    if (ticket && nvec <= kAmaxAloneBelow) return 1;
    const size_t chunk = (size_t)kThreads * (ticket && nvec < kAmaxSmallBelow ? kAmaxVecsSmall : kAmaxVecs), chunks = (nvec + chunk - 1) / chunk;
    const size_t most = ticket ? kAmaxBlocks : kAmaxAtomics;
    return (unsigned)(chunks < 1 ? 1 : chunks > most ? most : chunks);
}

// The work of workgroup `bid` of `grid` on one tensor.
template <int DT, bool TICKET>
__device__ __forceinline__ void amax_vec_body(const void* __restrict__ x, size_t n, unsigned* __restrict__ out_bits,
                                              unsigned* __restrict__ ws, int fmt, float* __restrict__ scale_out,
                                              unsigned bid, unsigned grid)
{
    constexpr int PV = Elem<DT>::per_vec;
    const u32x4_any* xv = (const u32x4_any*)x;
    const size_t nvec = n / PV;
    unsigned run[4] = {0u, 0u, 0u, 0u};
    if (TICKET && nvec > kThreads * kAmaxVecsSmall && nvec <= kAmaxAloneBelow) amax_chunks<DT, kAmaxVecsAlone>(xv, nvec, bid, grid, run);
    else if (TICKET && nvec < kAmaxSmallBelow) amax_chunks<DT, kAmaxVecsSmall>(xv, nvec, bid, grid, run);
    else amax_chunks<DT, kAmaxVecs>(xv, nvec, bid, grid, run);
    unsigned r;
    if (DT == FP8_F32) {
        const unsigned a = run[0] > run[1] ? run[0] : run[1], b = run[2] > run[3] ? run[2] : run[3];
        r = a > b ? a : b;
    } else {
        u16x2 p = __builtin_elementwise_max(
            __builtin_elementwise_max(__builtin_bit_cast(u16x2, run[0]), __builtin_bit_cast(u16x2, run[1])),
            __builtin_elementwise_max(__builtin_bit_cast(u16x2, run[2]), __builtin_bit_cast(u16x2, run[3])));
        unsigned short m = p.x > p.y ? p.x : p.y;
        r = (unsigned)m << 16;
    }
    if (bid == 0) {
        size_t t = nvec * PV + threadIdx.x;
        if (t < n) {
            unsigned m = scalar_mag<DT>(x, t);
            r = r > m ? r : m;
        }
    }
    r = block_max_u32(r);
    if (TICKET) {
        __syncthreads();                                    // block_max_u32's LDS cells are used again below
        amax_finish_ticket(r, ws, fmt, (float*)out_bits, scale_out, bid, grid);
        return;
    }
    // most workgroups find the cell already large enough and skip the atomic
    if (threadIdx.x == 0 && r > __hip_atomic_load(out_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out_bits, r);
}

template <int DT, bool TICKET>
__global__ __launch_bounds__(kThreads) void amax_vec_kernel(const void* __restrict__ x, size_t n,
                                                           unsigned* __restrict__ out_bits, unsigned* __restrict__ ws,
                                                           int fmt, float* __restrict__ scale_out)
{
    amax_vec_body<DT, TICKET>(x, n, out_bits, ws, fmt, scale_out, blockIdx.x, gridDim.x);
}

// Up to kMultiMax tensors in one launch (fp8_amax_scale_multi): the grid is the concatenation of the
// grids the single-tensor launches would use; tensor t has the workgroups first[t] .. first[t + 1] - 1,
// its own 4096 words of workspace, and cells t of amax_out / scale_out.
struct MultiTensors {
    const void* x[kMultiMax];
    uint8_t* q[kMultiMax];
    size_t n[kMultiMax];
    int fmt[kMultiMax];
    unsigned first[kMultiMax + 1];
    int count;
};

__device__ __forceinline__ int multi_find(const MultiTensors& m, unsigned b)
{
    int t = 0;
#pragma unroll
    for (int i = 1; i < kMultiMax; ++i)
        if (i < m.count && b >= m.first[i]) t = i;
    return t;
}

template <int DT>
__global__ __launch_bounds__(kThreads) void amax_multi_kernel(MultiTensors m, float* __restrict__ amax_out,
                                                             float* __restrict__ scale_out, unsigned* __restrict__ ws)
{
    const int t = multi_find(m, blockIdx.x);
    amax_vec_body<DT, true>(m.x[t], m.n[t], (unsigned*)(amax_out + t), ws + (size_t)t * (FP8_AMAX_WORKSPACE_BYTES / 4), m.fmt[t],
                            scale_out ? scale_out + t : nullptr, blockIdx.x - m.first[t], m.first[t + 1] - m.first[t]);
}

// n == 0 in the one-launch form: amax 0, scale by the degenerate rule.
__global__ void amax_empty_kernel(int fmt, float* __restrict__ amax_out, float* __restrict__ scale_out)
{
    *amax_out = 0.0f;
    if (scale_out) *scale_out = scale_rule(0.0f, fmt);
}

__global__ void scale_kernel(const float* __restrict__ amax, int fmt, float* __restrict__ out)
{
    *out = scale_rule(*amax, fmt);
}

// ------------------------------------------------------------------------------------------
// The cast.  y = fl32(x * scale) is one IEEE multiply; then y is rounded to the nearest
// FP8 value, ties to the even code (Table 1 encodings), finite overflow saturates to the
// largest finite value (Section 2), NaN -> NaN, inf -> NaN (E4M3) or inf (E5M2).
// ------------------------------------------------------------------------------------------

// x and q at any address.  Every workgroup owns one contiguous run of the
// tensor (see cast_run / cast_group for how its lanes share the work).  Stores are ordinary up to
// kStreamingStoreBytes of output, where they win 5 % because part of the output stays in the
// 256 MB memory-side cache, and non-temporal beyond (5-8 % better there).
template <int DT, int FMT, int PATH, bool NTS>
__device__ __forceinline__ void quantize_vec_body(const void* __restrict__ x, size_t n, float s, uint8_t* __restrict__ q,
                                                  unsigned bid, unsigned grid)
{
    constexpr int VPI = DT == FP8_BF16 ? 2 : 4;     // 16-byte vectors per 16 elements
    const size_t nitem = n / 16;
    const size_t per = (nitem + grid - 1) / grid;
    const size_t lo = (size_t)bid * per;
    const size_t hi = lo + per < nitem ? lo + per : nitem;
    unsigned unused = 0;
    if (lo < hi)
        cast_run<DT, FMT, PATH, NTS, false>((const u32x4_any*)x, (typename Piece<DT>::type*)q, VPI * lo, VPI * hi, s, unused);
    if (bid == 0) {                                 // fewer than 16 tail elements
        const size_t t = nitem * 16 + threadIdx.x;
        if (t < n) q[t] = (uint8_t)encode_bits<FMT, PATH != kCastBitsStrict>(load_scalar<DT>(x, t) * s);
    }
}

template <int DT, int FMT, int PATH, bool NTS>
__global__ __launch_bounds__(kThreads) void quantize_vec_kernel(const void* __restrict__ x, size_t n,
                                                               float scale,
                                                               const float* __restrict__ scale_dev,
                                                               uint8_t* __restrict__ q)
{
    quantize_vec_body<DT, FMT, PATH, NTS>(x, n, scale_dev ? *scale_dev : scale, q, blockIdx.x, gridDim.x);
}

// Up to kMultiMax tensors in one launch (fp8_quantize_multi), grid as for amax_multi_kernel; tensor t is
// cast with scale_dev[t] to format fmt[t].
template <int DT, int PATH>
__global__ __launch_bounds__(kThreads) void quantize_multi_kernel(MultiTensors m, const float* __restrict__ scale_dev)
{
    const int t = multi_find(m, blockIdx.x);
    const unsigned bid = blockIdx.x - m.first[t], grid = m.first[t + 1] - m.first[t];
    if (m.fmt[t] == FP8_E4M3) quantize_vec_body<DT, FP8_E4M3, PATH, false>(m.x[t], m.n[t], scale_dev[t], m.q[t], bid, grid);
    else quantize_vec_body<DT, FP8_E5M2, PATH, false>(m.x[t], m.n[t], scale_dev[t], m.q[t], bid, grid);
}

// ------------------------------------------------------------------------------------------
// amax, factor and cast of tensors that fit the chip's registers (up to kMultiMax of them) in ONE launch that reads them once
// (fp8_scaled_gemm).  Two launches cost what launches cost, on the host and
// between the kernels, and a second read; here a workgroup keeps its chunk in registers while the maxima of all
// chunks of the tensor meet in the workspace, and casts it from there:
//   - workgroup b leaves its maximum in slot b and reads the others until all are there.  A slot holds
//     the maximum with bit 31 set (maxima have it clear), so the value is its own flag: one store and
//     one load per lane of a wave, agent-scope atomics both, no other data is exchanged through memory;
//   - nobody has to be resident for anybody else to finish: a workgroup that has waited kCastPatience
//     sees to the maxima that are missing itself, with the others that wait (missing_maxima);
//   - the last workgroup to have read the slots clears them for the next call.
// Up to kMostChunks chunks of the size that the tensors need.  Measured, amax + cast of both operands, two launches -> one: 0.5 MB of fp32
// 6.9 -> 3.8 us, 1 MB of bf16 7.4 -> 5.0; whole steps 630 x 1472 x 640 (2.6 MB) 17.2 -> 14.3, 387 x 960 x 1920 (5 MB) 18.4 -> 15.7, 1092 x 1856 x
// 2624 (15 MB) 37.4 -> 35.7, 1638 x 704 x 6272 (28 MB) 50.4 -> 44.5; 90 steps from 2.5 to 39 MB all faster, by 2 to 25 %.
// The 1024-thread forms take a compute unit each, so two streams' launches, or one beside a long product, do not all run at once.  10 us is about
// twice what the maxima take on an empty chip; from 0.5 to 20 us a call took the same alone, on two and on four streams, with 70 us 5 - 25 % more on four.
// Four streams of such steps, two launches / one: 2048 x 4096 x 2048 161 / 177 us a call, 2048 x 6144 x 2048 240 / 245, 1638 x 704 x 6272 169 / 167,
// 2048 x 2000 x 2000 of fp32 134 / 136; two streams 89 / 80, 117 / 112, 90 / 78, 64 / 59; beside a product of a millisecond 440 / 427 (40 MB), 440 / 326 (17 MB).
// ------------------------------------------------------------------------------------------
constexpr unsigned kCastPatience = 1000;                             // 10 us
constexpr unsigned kMostChunks = 256;                                // of a launch, and no more than compute units: on an empty chip all workgroups run at once
static_assert((kCastSlots + kMostChunks) * sizeof(unsigned) <= FP8_AMAX_WORKSPACE_BYTES, "a slot per chunk");

// The vectors of chunk b that the thread holds (zeros where there are none), and its tail element if it has one
// (the elements behind the last whole vector belong to the last chunk): their largest magnitude.
template <int DT, int THREADS, int VECS>
__device__ __forceinline__ unsigned load_chunk(const void* x, size_t n, size_t b, bool tail, u32x4 (&v)[VECS])
{
    const u32x4_any* xv = (const u32x4_any*)x;
    const size_t nvec = n / Elem<DT>::per_vec;
    unsigned run = 0;
#pragma unroll
    for (int k = 0; k < VECS; ++k) {
        const size_t i = b * ((size_t)THREADS * VECS) + threadIdx.x + (size_t)k * THREADS;
        v[k] = (u32x4){0u, 0u, 0u, 0u};
        if (i < nvec) v[k] = xv[i];
    }
#pragma unroll
    for (int k = 0; k < VECS; ++k) run = vec_mag_max<DT>(v[k], run);
    const size_t t = nvec * Elem<DT>::per_vec + threadIdx.x;
    const unsigned r = run_to_bits<DT>(run);
    return tail && t < n ? max(r, scalar_mag<DT>(x, t)) : r;
}

template <int DT, int FMT, int THREADS, int VECS>
__device__ __forceinline__ void amax_cast_body(const void* __restrict__ x, size_t n, uint8_t* __restrict__ q, float* __restrict__ amax_out,
                                               float* __restrict__ scale_out, unsigned* __restrict__ ws, unsigned bid, unsigned grid, unsigned patience)
{
    constexpr int VPI = DT == FP8_BF16 ? 2 : 4;              // vectors that make 16 elements
    u32x4 v[VECS];
    const unsigned own = block_max_u32<THREADS>(load_chunk<DT, THREADS, VECS>(x, n, bid, bid == grid - 1, v));
    __shared__ unsigned largest;
    __shared__ unsigned long long absent[kMostChunks / 64];  // chunks whose maximum has not come
    __shared__ bool complete;                                // there are none
    unsigned ticket = 0;                                     // of the workgroup among the readers of the slots (first lane)
    if (threadIdx.x < 64) {
        const unsigned l = threadIdx.x;
        if (l == 0 && grid > 1) __hip_atomic_store(&ws[kCastSlots + bid], own | 0x80000000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long began = wall_clock64();
        unsigned m = own;
        unsigned long long any = 0;
        for (unsigned k = 0; 64 * k < grid; ++k) {
            const unsigned slot = 64 * k + l;
            unsigned p = slot < grid && grid > 1 ? 0u : 0x80000000u;
            while (!(p >> 31)) {
                p = __hip_atomic_load(&ws[kCastSlots + slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (wall_clock64() - began > patience) break;
            }
            m = max(m, p & 0x7fffffffu);
            const unsigned long long gone = ~__ballot(p >> 31);
            any |= gone;
            if (l == 0) absent[k] = gone;
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0x0070);                  // vmcnt(0): the own maximum has been acknowledged
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        m = wave_max_u32(m);
        if (l == 0) {
            largest = m;
            complete = any == 0;
            // (nobody waits for the answer before the end: waited for here it was 0.8 us of every workgroup's time)
            if (grid > 1 && any == 0) ticket = __hip_atomic_fetch_add(&ws[kCastDone], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (__builtin_expect(!complete, 0)) {                    // (never, unless other work held compute units for as long)
        missing_maxima(absent, grid, bid, [&](unsigned i) { return &ws[kCastSlots + i]; },
                       [&](unsigned i) {
                           u32x4 other[VECS];
                           return block_max_u32<THREADS>(load_chunk<DT, THREADS, VECS>(x, n, i, i == grid - 1, other));
                       },
                       [&](unsigned, unsigned m) { atomicMax(&largest, m); });
        if (threadIdx.x == 0) {
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0): the maxima of others have been acknowledged
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            ticket = __hip_atomic_fetch_add(&ws[kCastDone], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    const float a = as_f32(largest), s = scale_rule(a, FMT);
    if (bid == 0 && threadIdx.x == 0) { *amax_out = a; *scale_out = s; }
    const size_t nvec = n / Elem<DT>::per_vec, first = bid * ((size_t)THREADS * VECS) + threadIdx.x;
    typename Piece<DT>::type* qp = (typename Piece<DT>::type*)q;
#pragma unroll
    for (int g = 0; g < VECS / VPI; ++g) {
        u32x4 item[VPI];
        float y[16];
#pragma unroll
        for (int k = 0; k < VPI; ++k) item[k] = v[g * VPI + k];
        scale_item<DT>(item, s, y);
        const u32x4 o = encode16<FMT, kCastCvt>(y);
#pragma unroll
        for (int k = 0; k < VPI; ++k) {
            const size_t i = first + (size_t)(g * VPI + k) * THREADS;
            if (i < nvec) qp[i] = Piece<DT>::of(o, k);
        }
    }
    const size_t t = nvec * Elem<DT>::per_vec + threadIdx.x;
    if (bid == grid - 1 && t < n) q[t] = (uint8_t)encode_bits<FMT>(load_scalar<DT>(x, t) * s);
    if (threadIdx.x < 64 && grid > 1 && (unsigned)__builtin_amdgcn_readfirstlane((int)ticket) == grid - 1) {
        for (unsigned i = threadIdx.x; i < grid; i += 64) __hip_atomic_store(&ws[kCastSlots + i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (threadIdx.x == 0) __hip_atomic_store(&ws[kCastDone], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int DT, int THREADS, int VECS>
__global__ __launch_bounds__(THREADS) void amax_cast_kernel(MultiTensors m, float* __restrict__ amax_out, float* __restrict__ scale_out,
                                                                unsigned* __restrict__ ws, unsigned patience)
{
    const int t = multi_find(m, blockIdx.x);
    const unsigned bid = blockIdx.x - m.first[t], grid = m.first[t + 1] - m.first[t];
    unsigned* w = ws + (size_t)t * (FP8_AMAX_WORKSPACE_BYTES / 4);
    if (m.fmt[t] == FP8_E4M3) amax_cast_body<DT, FP8_E4M3, THREADS, VECS>(m.x[t], m.n[t], m.q[t], amax_out + t, scale_out + t, w, bid, grid, patience);
    else amax_cast_body<DT, FP8_E5M2, THREADS, VECS>(m.x[t], m.n[t], m.q[t], amax_out + t, scale_out + t, w, bid, grid, patience);
}

}  // namespace

namespace {
// ws == nullptr: amax_out was cleared by the caller, workgroups raise it with atomics.
// ws != nullptr: the one-launch form (see amax_finish_ticket); grids stay within kAmaxBlocks.
template <bool TICKET>
void launch_amax_kernels(const void* x, size_t n, int in_dtype, unsigned* out, unsigned* ws, int fmt, float* scale_out,
                         hipStream_t stream)
{
    const unsigned grid = amax_grid(n / (in_dtype == FP8_F32 ? 4 : 8), TICKET);
    if (in_dtype == FP8_F32)
        enqueue((amax_vec_kernel<FP8_F32, TICKET>), dim3(grid), dim3(kThreads), 0, stream, x, n, out, ws, fmt, scale_out);
    else
        enqueue((amax_vec_kernel<FP8_BF16, TICKET>), dim3(grid), dim3(kThreads), 0, stream, x, n, out, ws, fmt, scale_out);
}
}  // namespace

int launch_amax(const void* x, size_t n, int in_dtype, float* amax_out, hipStream_t stream)
{
    unsigned* out = (unsigned*)amax_out;
    enqueue(store_u32_kernel, dim3(1), dim3(1), 0, stream, out, 0u);
    if (n == 0) return check_launch("amax init");
    launch_amax_kernels<false>(x, n, in_dtype, out, nullptr, 0, nullptr, stream);
    return check_launch("amax");
}

int launch_amax_scale(const void* x, size_t n, int in_dtype, int fmt, float* amax_out, float* scale_out, void* workspace,
                      hipStream_t stream)
{
    static_assert((kTicketPartials + kAmaxBlocks) * sizeof(unsigned) <= FP8_AMAX_WORKSPACE_BYTES, "counters + one partial per workgroup");
    if (n == 0) enqueue(amax_empty_kernel, dim3(1), dim3(1), 0, stream, fmt, amax_out, scale_out);
    else launch_amax_kernels<true>(x, n, in_dtype, (unsigned*)amax_out, (unsigned*)workspace, fmt, scale_out, stream);
    return check_launch("amax_scale");
}

// One launch where no tensor is empty; tensor by tensor otherwise.  Results are those of the single-tensor launches either way.
int launch_amax_scale_multi(int count, const void* const* x, const size_t* n, int in_dtype, const int* fmt, float* amax_out,
                            float* scale_out, void* workspace, hipStream_t stream)
{
    bool one = count > 1;
    for (int i = 0; i < count; ++i) one = one && n[i] > 0;
    if (!one) {
        for (int i = 0; i < count; ++i)
            if (int e = launch_amax_scale(x[i], n[i], in_dtype, fmt[i], amax_out + i, scale_out ? scale_out + i : nullptr,
                                          (char*)workspace + (size_t)i * FP8_AMAX_WORKSPACE_BYTES, stream))
                return e;
        return FP8_OK;
    }
    MultiTensors m{};
    m.count = count;
    unsigned total = 0;
    const size_t per_vec = in_dtype == FP8_F32 ? 4 : 8;
    for (int i = 0; i < count; ++i) {
        m.x[i] = x[i]; m.n[i] = n[i]; m.fmt[i] = fmt[i]; m.first[i] = total;
        total += amax_grid(n[i] / per_vec, true);
    }
    for (int i = count; i <= kMultiMax; ++i) m.first[i] = total;
    if (in_dtype == FP8_F32)
        enqueue(amax_multi_kernel<FP8_F32>, dim3(total), dim3(kThreads), 0, stream, m, amax_out, scale_out, (unsigned*)workspace);
    else
        enqueue(amax_multi_kernel<FP8_BF16>, dim3(total), dim3(kThreads), 0, stream, m, amax_out, scale_out, (unsigned*)workspace);
    return check_launch("amax_scale_multi");
}

float scale_from_amax_host(float amax, int fmt) { return scale_rule(amax, fmt); }

int launch_scale_from_amax(const float* amax, int fmt, float* scale_out, hipStream_t stream)
{
    enqueue(scale_kernel, dim3(1), dim3(1), 0, stream, amax, fmt, scale_out);
    return check_launch("scale_from_amax");
}

namespace {
// Workgroups of the cast kernels: runs of 4 items of 16 elements per lane (the knob FP8_KNOB_CAST_RUN
// overrides), shorter ones where that would leave the chip with fewer than 512 workgroups (1024 for
// fp32, whose items are twice as long: 8.4 10^6 elements 27.9 -> 24.6 us with the other steps of a cast).
int cast_grid(size_t n, int in_dtype)
{
    const size_t items = n / 16, spread = items / ((size_t)kThreads * (in_dtype == FP8_F32 ? 1024 : 512));
    const size_t per_lane = knob(FP8_KNOB_CAST_RUN) ? (size_t)knob(FP8_KNOB_CAST_RUN) : spread < 1 ? 1 : spread > 4 ? 4 : spread;
    return grid_for((items + per_lane - 1) / per_lane, kCastBlocks);
}

template <int DT, int FMT>
void launch_quantize_typed(const void* x, size_t n, float scale, const float* scale_dev,
                           uint8_t* q, bool saturate, hipStream_t stream)
{
    const int grid = cast_grid(n, DT);
    // An output that does not fit the memory-side cache (256 MB) is written past it.
    const bool nts = n >= kStreamingStoreBytes;
#define FP8MM_LAUNCH_QV(PATH)                                                                                      \
    do {                                                                                                           \
        if (nts) enqueue((quantize_vec_kernel<DT, FMT, PATH, true>), dim3(grid), dim3(kThreads), 0,     \
                                    stream, x, n, scale, scale_dev, q);                                            \
        else enqueue((quantize_vec_kernel<DT, FMT, PATH, false>), dim3(grid), dim3(kThreads), 0,        \
                                stream, x, n, scale, scale_dev, q);                                                \
    } while (0)
    if (!saturate) FP8MM_LAUNCH_QV(kCastBitsStrict);
    else if (cast_path() == kCastCvt) FP8MM_LAUNCH_QV(kCastCvt);
    else FP8MM_LAUNCH_QV(kCastBits);
#undef FP8MM_LAUNCH_QV
}

// ------------------------------------------------------------------------------------------
// dequantize: out[i] = fl_out(decode(q[i]) / scale), one IEEE single division per element
// (Section 2: values are unscaled by the inverse of the scaling factor after conversion from
// FP8), then rounding to bf16 if asked.  16 bytes in, 32 or 64 bytes out per lane.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned to_bf16_bits(float f)
{
    const unsigned u = as_u32(f);
    const unsigned r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    return (u & 0x7fffffffu) > 0x7f800000u ? ((u >> 16) | 0x40u) : r;
}

template <int FMT, int OUT>
__global__ __launch_bounds__(kThreads) void dequantize_kernel(const uint8_t* __restrict__ q, size_t n, float scale,
                                                             const float* __restrict__ scale_dev,
                                                             void* __restrict__ out)
{
    // The result depends on the byte alone: every workgroup first tabulates the 256 results (one
    // decode, one IEEE division and, for bf16, one rounding per thread) in LDS, then streams.  With
    // the arithmetic done per element the kernel was bound by the vector ALU at 3.2 TB/s.
    // A lane takes the 8 (bf16 out) or 4 (fp32 out) bytes that make one 16-byte output vector, so that
    // the load and the store instruction of a wave both cover consecutive bytes.
    constexpr int EPV = OUT == FP8_F32 ? 4 : 8;
    constexpr int U = 4;                            // vectors per lane in flight
    static_assert(kThreads == 256, "one table entry per thread");
    __shared__ unsigned table[256];                 // fp32 bits, or bf16 bits in the low half
    {
        const float y = decode_fp8<FMT>(threadIdx.x) / (scale_dev ? *scale_dev : scale);
        table[threadIdx.x] = OUT == FP8_F32 ? as_u32(y) : to_bf16_bits(y);
    }
    __syncthreads();
    const size_t stride = (size_t)gridDim.x * kThreads;
    const size_t nvec = n / EPV;
    auto load_piece = [&](size_t i) {
        if (OUT == FP8_F32) return (u32x2){__builtin_nontemporal_load(&((const u32_any*)q)[i]), 0u};
        return (u32x2)__builtin_nontemporal_load(&((const u32x2_any*)q)[i]);
    };
    auto emit = [&](size_t i, u32x2 p) {
        unsigned r[EPV];
#pragma unroll
        for (int e = 0; e < EPV; ++e) r[e] = table[(p[e >> 2] >> (8 * (e & 3))) & 0xffu];
        u32x4 o;
        if constexpr (OUT == FP8_F32) {
            o = (u32x4){r[0], r[1], r[2], r[3]};
        } else {
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d] = r[2 * d] | (r[2 * d + 1] << 16);
        }
        ((u32x4_any*)out)[i] = o;
    };
    // every workgroup owns one contiguous run of the vectors
    const size_t per = (nvec + gridDim.x - 1) / gridDim.x;
    const size_t lo = (size_t)blockIdx.x * per;
    const size_t hi = lo + per < nvec ? lo + per : nvec;
    size_t i = lo + threadIdx.x;
    for (; i + (U - 1) * kThreads < hi; i += U * kThreads) {
        u32x2 p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) p[u] = load_piece(i + u * kThreads);
#pragma unroll
        for (int u = 0; u < U; ++u) emit(i + u * kThreads, p[u]);
    }
    for (; i < hi; i += kThreads) emit(i, load_piece(i));
    for (size_t t = nvec * EPV + (size_t)blockIdx.x * kThreads + threadIdx.x; t < n; t += stride) {
        if (OUT == FP8_F32) ((unsigned*)out)[t] = table[q[t]];
        else ((unsigned short*)out)[t] = (unsigned short)table[q[t]];
    }
}
}  // namespace

int launch_quantize(const void* x, size_t n, int in_dtype, int fmt, float scale,
                    const float* scale_dev, bool saturate, uint8_t* q_out, hipStream_t stream)
{
    if (n == 0) return FP8_OK;
    if (in_dtype == FP8_F32) {
        if (fmt == FP8_E4M3) launch_quantize_typed<FP8_F32, FP8_E4M3>(x, n, scale, scale_dev, q_out, saturate, stream);
        else                 launch_quantize_typed<FP8_F32, FP8_E5M2>(x, n, scale, scale_dev, q_out, saturate, stream);
    } else {
        if (fmt == FP8_E4M3) launch_quantize_typed<FP8_BF16, FP8_E4M3>(x, n, scale, scale_dev, q_out, saturate, stream);
        else                 launch_quantize_typed<FP8_BF16, FP8_E5M2>(x, n, scale, scale_dev, q_out, saturate, stream);
    }
    return check_launch("quantize");
}

int launch_dequantize(const uint8_t* q, size_t n, int fmt, float scale, const float* scale_dev,
                      int out_dtype, void* out, hipStream_t stream)
{
    if (n == 0) return FP8_OK;
    const int grid = grid_for(n / 16 + 1, 256 * 256);     // many short runs measured best (write-heavy stream)
    if (fmt == FP8_E4M3) {
        if (out_dtype == FP8_F32) enqueue((dequantize_kernel<FP8_E4M3, FP8_F32>), dim3(grid), dim3(kThreads), 0, stream, q, n, scale, scale_dev, out);
        else enqueue((dequantize_kernel<FP8_E4M3, FP8_BF16>), dim3(grid), dim3(kThreads), 0, stream, q, n, scale, scale_dev, out);
    } else {
        if (out_dtype == FP8_F32) enqueue((dequantize_kernel<FP8_E5M2, FP8_F32>), dim3(grid), dim3(kThreads), 0, stream, q, n, scale, scale_dev, out);
        else enqueue((dequantize_kernel<FP8_E5M2, FP8_BF16>), dim3(grid), dim3(kThreads), 0, stream, q, n, scale, scale_dev, out);
    }
    return check_launch("dequantize");
}

int launch_quantize_multi(int count, const void* const* x, const size_t* n, int in_dtype, const int* fmt,
                          const float* scale_dev, uint8_t* const* q_out, hipStream_t stream)
{
    // one launch where no tensor is empty and all take ordinary stores; else tensor by tensor
    bool one = count > 1;
    for (int i = 0; i < count; ++i) one = one && n[i] > 0 && n[i] < kStreamingStoreBytes;
    if (!one) {
        for (int i = 0; i < count; ++i)
            if (int e = launch_quantize(x[i], n[i], in_dtype, fmt[i], 0.0f, scale_dev + i, true, q_out[i], stream)) return e;
        return FP8_OK;
    }
    MultiTensors m{};
    m.count = count;
    unsigned total = 0;
    for (int i = 0; i < count; ++i) {
        m.x[i] = x[i]; m.q[i] = q_out[i]; m.n[i] = n[i]; m.fmt[i] = fmt[i]; m.first[i] = total;
        total += (unsigned)cast_grid(n[i], in_dtype);
    }
    for (int i = count; i <= kMultiMax; ++i) m.first[i] = total;
    const bool cvt = cast_path() == kCastCvt;
    if (in_dtype == FP8_F32) {
        if (cvt) enqueue((quantize_multi_kernel<FP8_F32, kCastCvt>), dim3(total), dim3(kThreads), 0, stream, m, scale_dev);
        else enqueue((quantize_multi_kernel<FP8_F32, kCastBits>), dim3(total), dim3(kThreads), 0, stream, m, scale_dev);
    } else {
        if (cvt) enqueue((quantize_multi_kernel<FP8_BF16, kCastCvt>), dim3(total), dim3(kThreads), 0, stream, m, scale_dev);
        else enqueue((quantize_multi_kernel<FP8_BF16, kCastBits>), dim3(total), dim3(kThreads), 0, stream, m, scale_dev);
    }
    return check_launch("quantize_multi");
}

// The forms of the one-launch amax + cast: workgroup and vectors of 16 bytes per lane, which make a chunk of 64, 128 or 160 KB.  (With more
// vectors a lane's registers went to scratch memory, and operands of 48 to 64 MB took 3 to 10 % longer than in two launches.)
constexpr struct { int threads, vecs; } kCastForm[] = {{512, 8}, {1024, 8}, {1024, 10}};
constexpr int kCastForms = 3;

// amax, factors and casts of `count` tensors: one launch where the tensors fit (see amax_cast_kernel), else
// the two launches of the multi-tensor forms.
int launch_amax_cast(int count, const void* const* x, const size_t* n, int in_dtype, const int* fmt, float* amax_out, float* scale_out,
                     void* workspace, uint8_t* const* q_out, hipStream_t stream)
{
    const size_t per_vec = in_dtype == FP8_F32 ? 4 : 8;
    bool one = cast_path() == kCastCvt;
    for (int i = 0; i < count; ++i) one = one && n[i] > 0;
    auto chunks_of = [&](int i, size_t vecs) { return std::max<size_t>(1, (n[i] / per_vec + vecs - 1) / vecs); };
    auto chunks = [&](size_t vecs) { size_t c = 0; for (int i = 0; i < count; ++i) c += chunks_of(i, vecs); return c; };
    const size_t most = std::min<size_t>(kMostChunks, compute_units());
    int form = -1;
    if (one)
        for (int f = 0; f < kCastForms && form < 0; ++f)
            if (kCastForm[f].vecs % (in_dtype == FP8_F32 ? 4 : 2) == 0 && chunks((size_t)kCastForm[f].threads * kCastForm[f].vecs) <= most) form = f;
    if (form < 0) {
        if (int e = launch_amax_scale_multi(count, x, n, in_dtype, fmt, amax_out, scale_out, workspace, stream)) return e;
        return launch_quantize_multi(count, x, n, in_dtype, fmt, scale_out, q_out, stream);
    }
    MultiTensors m{};
    m.count = count;
    unsigned total = 0;
    const size_t chunk = (size_t)kCastForm[form].threads * kCastForm[form].vecs;
    for (int i = 0; i < count; ++i) {
        m.x[i] = x[i]; m.q[i] = q_out[i]; m.n[i] = n[i]; m.fmt[i] = fmt[i]; m.first[i] = total;
        total += (unsigned)chunks_of(i, chunk);
    }
    for (int i = count; i <= kMultiMax; ++i) m.first[i] = total;
    const unsigned ticks = patience(kCastPatience);
    unsigned* ws = (unsigned*)workspace;
#define FP8MM_LAUNCH_CAST(DT, THREADS, VECS) \
    enqueue((amax_cast_kernel<DT, THREADS, VECS>), dim3(total), dim3(THREADS), 0, stream, m, amax_out, scale_out, ws, ticks)
    if (in_dtype == FP8_F32) {
        if (form == 0) FP8MM_LAUNCH_CAST(FP8_F32, 512, 8); else FP8MM_LAUNCH_CAST(FP8_F32, 1024, 8);
    } else {
        if (form == 0) FP8MM_LAUNCH_CAST(FP8_BF16, 512, 8);
        else if (form == 1) FP8MM_LAUNCH_CAST(FP8_BF16, 1024, 8);
        else FP8MM_LAUNCH_CAST(FP8_BF16, 1024, 10);
    }
#undef FP8MM_LAUNCH_CAST
    return check_launch("amax_cast");
}

}  // namespace fp8mm
