// Device helpers shared by the gfx950 kernels: vector loads of caller-owned gradient rows
// of any alignment, wavefront reductions with a fixed tree, and the AMSGrad update line.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <type_traits>

#include "launch_rules.h"

namespace cams {

// Which tile a workgroup works on.  The hardware hands the workgroups of a launch to the chip's eight XCDs in
// turn (linear workgroup id modulo 8), so with tile = block id every XCD walks over every page of a row.  With
// chunk > 0 the blocks are taken in groups of 8 * chunk, and inside a group XCD x works through the contiguous
// tiles [x * chunk, (x + 1) * chunk) of the group.  Such a grid has a multiple of 8 * chunk blocks in x
// (grid_blocks); blocks whose tile is past the last one leave at once.  chunk = 0: tile = block id.
__device__ __forceinline__ int tile_of_block(unsigned b, int chunk)
{
    if (chunk <= 0) return (int)b;
    const unsigned span = 8u * (unsigned)chunk, within = b % span;
    return (int)(b - within + (within & 7u) * (unsigned)chunk + (within >> 3));
}

constexpr int kWave = 64;          // CDNA wavefront
constexpr int kThreads = 256;      // workgroup size of every streaming kernel (4 waves)
constexpr int kTile = 4096;        // coordinates per tile; rows of library-owned arrays are padded to it

// fp32 operations with one IEEE rounding each.  The translation unit is built with
// -ffp-contract=off and the pragma below repeats it, so a*b+c is never fused; `/` and sqrtf are
// the correctly rounded forms (hipcc's default for fp32; the __fsqrt_rn intrinsic is NOT: it maps
// to the approximate native square root).
#pragma clang fp contract(off)
__device__ __forceinline__ float fadd(float a, float b) { return a + b; }
__device__ __forceinline__ float fsub(float a, float b) { return a - b; }
__device__ __forceinline__ float fmul(float a, float b) { return a * b; }
__device__ __forceinline__ float fdiv(float a, float b) { return a / b; }
__device__ __forceinline__ float fsqrt(float a) { return sqrtf(a); }

// Hyper-parameters of the AMSGrad recursion (Section 3), fp32, prepared on the host.
struct AmsParams {
    float beta1, beta2, omb1, omb2;   // omb = 1 - beta, rounded once to fp32
    float eps, lr;
    int32_t eps_mode;                 // 0: sqrt(vhat)+eps   1: sqrt(vhat+eps)
    float n_workers;                  // divisor of the server average
    int32_t stream_state;             // theta, m, v, vhat are loaded and stored as streams (non-temporal): the host
                                      // launches the kStreamState = true variants of the update kernels
};

// m, v, vhat, theta update on one coordinate; every operation rounds to fp32 on its own
// (no fused multiply-add).
__device__ __forceinline__ void amsgrad_update(float &theta, float &m, float &v, float &vhat, float gbar,
                                               const AmsParams &p)
{
    m = fadd(fmul(p.beta1, m), fmul(p.omb1, gbar));
    v = fadd(fmul(p.beta2, v), fmul(p.omb2, fmul(gbar, gbar)));
    vhat = fmaxf(vhat, v);
    float den = p.eps_mode ? fsqrt(fadd(vhat, p.eps)) : fadd(fsqrt(vhat), p.eps);
    theta = fsub(theta, fdiv(fmul(p.lr, m), den));
}

__device__ __forceinline__ void amsgrad_update4(float4 &th, float4 &m, float4 &v, float4 &vh, const float4 &g,
                                                const AmsParams &p)
{
    amsgrad_update(th.x, m.x, v.x, vh.x, g.x, p);
    amsgrad_update(th.y, m.y, v.y, vh.y, g.y, p);
    amsgrad_update(th.z, m.z, v.z, vh.z, g.z, p);
    amsgrad_update(th.w, m.w, v.w, vh.w, g.w, p);
}

typedef float v4f __attribute__((ext_vector_type(4)));

// Vector types of a lower alignment: gfx950 takes a global load of 8 or 16 bytes at any address, so a row that
// starts between two 16-byte boundaries is still read with one wide load per lane.  A wavefront's 1 KB then
// touches nine 128-byte lines instead of eight, where 4- and 8-byte loads of the same data took two to four times
// the load instructions.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t v2u_any __attribute__((ext_vector_type(2), aligned(2)));

// Streaming (read-once) loads: the gradient is never read again by the same step.  p: 4-byte aligned.
__device__ __forceinline__ float4 stream_load4(const float *p)
{
    const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f_any *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}

// Gradients come as fp32, as bfloat16 (the upper 16 bits of the fp32 value) or as IEEE half precision.  16-bit values are
// widened exactly, so every formula downstream sees the same fp32 numbers as with an fp32 copy of them.
struct f16bits {          // only tells the two 16-bit formats apart
    uint16_t v;
};
static_assert(sizeof(f16bits) == 2, "f16bits is a plain 16-bit value");

typedef uint32_t v2u __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float bf16_to_float(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ float f16_to_float(uint32_t h) { return __half2float(__ushort_as_half((unsigned short)h)); }

// Four consecutive gradient coordinates row[j..j+3] as they stand in memory, j a multiple of 4, and their fp32 values.
// The row is caller memory of length d at any alignment of its element type (row i of a dense [n][d] array starts
// at i*d elements); coordinates at or beyond d read as zero.  kInside: j + 4 <= d is known.
// Loading and widening are apart so that a thread's loads all go out before it waits for the first: widened inside the
// bounds check, each 16-bit load was waited for before the next was issued.
template <typename G> struct GradRaw { v2u v; };
template <> struct GradRaw<float> { v4f v; };

template <bool kInside>
__device__ __forceinline__ GradRaw<float> load_raw4(const float *__restrict__ row, int64_t j, int64_t d)
{
    const float *p = row + j;
    if (kInside || j + 4 <= d) return {__builtin_nontemporal_load(reinterpret_cast<const v4f_any *>(p))};
    v4f r = {0.f, 0.f, 0.f, 0.f};
    if (j < d) r.x = p[0];
    if (j + 1 < d) r.y = p[1];
    if (j + 2 < d) r.z = p[2];
    if (j + 3 < d) r.w = p[3];
    return {r};
}
template <bool kInside, typename G>   // G: uint16_t (bfloat16 bits) or f16bits
__device__ __forceinline__ GradRaw<G> load_raw4(const G *__restrict__ row, int64_t j, int64_t d)
{
    const uint16_t *p = reinterpret_cast<const uint16_t *>(row) + j;
    if (kInside || j + 4 <= d) return {__builtin_nontemporal_load(reinterpret_cast<const v2u_any *>(p))};
    v2u r = {0u, 0u};
    if (j < d) r.x = p[0];
    if (j + 1 < d) r.x |= (uint32_t)p[1] << 16;
    if (j + 2 < d) r.y = p[2];
    if (j + 3 < d) r.y |= (uint32_t)p[3] << 16;
    return {r};
}
// The same without a branch, for d >= 4: a float4 that ends past d is read from the row's last four coordinates and shifted, so
// that the loads of several rows go out together whatever the lane (a branch around a load that ends early waits for the loads
// before it).
struct GradPlace {
    int64_t at;      // where the four are read: j, or d - 4
    int shift;       // j - at, no more than 4
};
__device__ __forceinline__ GradPlace grad_place(int64_t j, int64_t d)
{
    const int64_t at = min(j, d - 4);
    return {at, (int)min(j - at, (int64_t)4)};
}
__device__ __forceinline__ GradRaw<float> load_place4(const float *__restrict__ row, const GradPlace &q)
{
    return {__builtin_nontemporal_load(reinterpret_cast<const v4f_any *>(row + q.at))};
}
template <typename G>
__device__ __forceinline__ GradRaw<G> load_place4(const G *__restrict__ row, const GradPlace &q)
{
    return {__builtin_nontemporal_load(reinterpret_cast<const v2u_any *>(reinterpret_cast<const uint16_t *>(row) + q.at))};
}
// Components past d come out as anything.
__device__ __forceinline__ float4 shift4(float4 x, int shift)
{
    if (shift & 1) x = make_float4(x.y, x.z, x.w, x.w);
    if (shift & 2) x = make_float4(x.z, x.w, x.w, x.w);
    return x;
}
__device__ __forceinline__ float4 widen4(const GradRaw<float> &r) { return make_float4(r.v.x, r.v.y, r.v.z, r.v.w); }
__device__ __forceinline__ float4 widen4(const GradRaw<uint16_t> &r)
{
    return make_float4(__uint_as_float(r.v.x << 16), __uint_as_float(r.v.x & 0xffff0000u), __uint_as_float(r.v.y << 16),
                       __uint_as_float(r.v.y & 0xffff0000u));
}
__device__ __forceinline__ float4 widen4(const GradRaw<f16bits> &r)
{
    return make_float4(f16_to_float(r.v.x & 0xffffu), f16_to_float(r.v.x >> 16), f16_to_float(r.v.y & 0xffffu),
                       f16_to_float(r.v.y >> 16));
}

// base + at for a base that is uniform over the wavefront: the offset stays a 32-bit number of bytes (at * sizeof(T) < 2^32), so that
// the access takes it beside a scalar base instead of a 64-bit sum per lane.
template <typename T>
__device__ __forceinline__ T *at_offset(T *base, uint32_t at)
{
    using Bytes = std::conditional_t<std::is_const<T>::value, const char, char>;
    return reinterpret_cast<T *>(reinterpret_cast<Bytes *>(base) + offset_bytes(at, (uint32_t)sizeof(T)));
}

__device__ __forceinline__ float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ void st4(float *p, const float4 &v) { *reinterpret_cast<float4 *>(p) = v; }

// Streaming (write-once) store: what a step writes to the stored rows and to theta, m, v, vhat is not
// read again before the next step.  Marking these accesses (and the matching loads) non-temporal keeps
// them from displacing what the step does reuse - candidates, sign words, scales - and measured 7 - 11 %
// off the whole step on the large workloads.
__device__ __forceinline__ void st4_stream(float *p, const float4 &v)
{
    const v4f t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<v4f *>(p));
}
// A stored row (error memory / Markov sequence) is read once per step.  Rows that together are far
// larger than the caches cannot survive from one step to the next, so they are loaded as a stream; small
// ones (stream == 0) are loaded normally, since part of them is still cached from the step before.  (They
// are stored as a stream in both cases: that measured faster or equal at every size.)
// kApart: empty asm statements keep the two loads apart where the compiler would merge them into one without the hint.
template <bool kApart = false>
__device__ __forceinline__ float4 ld4_row(const float *p, int stream)
{
    if (!kApart) return stream ? stream_load4(p) : ld4(p);
    float4 v;
    if (stream) {
        asm volatile("");
        v = stream_load4(p);
        asm volatile("");
    } else {
        v = ld4(p);
    }
    return v;
}
// theta, m, v, vhat are read and written once per step: streamed when they are too large to stay in the
// memory-side cache until the next step (AmsParams::stream_state).
// A compile-time choice: with a run-time flag the compiler merges the two stores and drops the hint.
template <bool kStream>
__device__ __forceinline__ float4 ld4_state(const float *p)
{
    if constexpr (kStream) return stream_load4(p); else return ld4(p);
}
template <bool kStream>
__device__ __forceinline__ void st4_state(float *p, const float4 &v)
{
    if constexpr (kStream) st4_stream(p, v); else st4(p, v);
}

// st4_state (kStream) or st4, unless the location already holds v: `old` is what this thread loaded from p.  Skipping such a
// store leaves memory as it is, so results are the same bit for bit.  Lanes that share a line of kLineLanes * 16
// bytes decide together, so that a line is written whole or not at all.  All lanes of the wavefront must call
// this together (it uses a ballot).
constexpr int kLineLanes = 8;
template <bool kStream>
__device__ __forceinline__ void st4_if_changed(float *p, const float4 &v, const float4 &old)
{
    const bool changed = __float_as_uint(v.x) != __float_as_uint(old.x) || __float_as_uint(v.y) != __float_as_uint(old.y) ||
                         __float_as_uint(v.z) != __float_as_uint(old.z) || __float_as_uint(v.w) != __float_as_uint(old.w);
    const uint64_t b = __ballot(changed);
    const int lane = threadIdx.x & (kWave - 1);
    if ((b >> (lane & ~(kLineLanes - 1))) & ((1ull << kLineLanes) - 1ull)) st4_state<kStream>(p, v);
}

__device__ __forceinline__ uint32_t mag_key(float x) { return __float_as_uint(x) & 0x7fffffffu; }

// A workgroup barrier that orders LDS only: unlike __syncthreads it does not wait for stores to memory that are in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Sum over lanes 0 .. this one, by the lane permutes that ride in a vector instruction (a row of 16 lanes in four steps, then the
// rows before): six __shfl_up are six round trips through the LDS unit, one after the other.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);      // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);      // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);      // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);      // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);      // row_bcast:31 into rows 2 and 3
    return (uint32_t)x;
}
// The sum over all 64 lanes, uniform, from wave_scan's result.
__device__ __forceinline__ uint32_t scan_total(uint32_t scan) { return (uint32_t)__builtin_amdgcn_readlane((int)scan, kWave - 1); }

// Sum over the 64 lanes with a fixed butterfly; every lane receives the same result, and the
// result depends only on the lane values, not on timing.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Sum over a 256-thread workgroup in a fixed order; valid in every thread.  `scratch` holds
// at least 4 doubles of LDS.  Contains two barriers.
__device__ __forceinline__ double block_sum(double v, double *scratch)
{
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) scratch[wave] = v;
    __syncthreads();
    return ((scratch[0] + scratch[1]) + scratch[2]) + scratch[3];
}

// Plain streaming copy, 16 bytes per lane, four independent loads per thread, one 16 KB piece per
// workgroup, non-temporal on both sides: the yardstick for the HBM counters (it moves exactly the bytes it
// is given) and for the bandwidth a simple kernel reaches on this chip.  chunk: tile_of_block's, over the
// pieces; blocks past the last piece do nothing.
__global__ __launch_bounds__(kThreads) void probe_copy(float *__restrict__ dst, const float *__restrict__ src,
                                                       int64_t vecs, int chunk)
{
    const int64_t q0 = (int64_t)tile_of_block(blockIdx.x, chunk) * (4 * kThreads) + threadIdx.x;
    float4 v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (q0 + r * kThreads < vecs) v[r] = stream_load4(src + 4 * (q0 + r * kThreads));
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (q0 + r * kThreads < vecs) st4_stream(dst + 4 * (q0 + r * kThreads), v[r]);
}

// State handed to a caller in device memory: probe_copy's shape for any count and a destination of 4-byte alignment (src
// 16-byte aligned).  HBM-bound: d = 110 M, 440 MB read and written in 138 us, where the runtime's copy takes 172.  kStream:
// src is read as a stream (see the host code).
template <bool kStream>
__global__ __launch_bounds__(kThreads) void copy_out_floats(float *__restrict__ dst, const float *__restrict__ src,
                                                            int64_t count, int chunk)
{
    const int64_t j0 = 4 * ((int64_t)tile_of_block(blockIdx.x, chunk) * (4 * kThreads) + threadIdx.x);
    float4 v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (j0 + 4 * kThreads * r + 4 <= count) v[r] = ld4_state<kStream>(src + j0 + 4 * kThreads * r);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + 4 * kThreads * r;
        if (j + 4 <= count) {
            const v4f t = {v[r].x, v[r].y, v[r].z, v[r].w};
            __builtin_nontemporal_store(t, reinterpret_cast<v4f_any *>(dst + j));
        } else {
            for (int64_t q = j; q < count; ++q) dst[q] = src[q];     // fewer than four are left
        }
    }
}

// The access pattern of the streaming passes with nothing else: x[i][j] = x[i][j] + g[i][j] in place, rows of d
// floats (d a multiple of 4, rows 16-byte aligned), one 16 KB piece of a row per workgroup, non-temporal on all
// three streams.  What this reaches is the practical ceiling for a kernel that reads two arrays and writes one of
// them back on this chip; the passes are measured against it.  chunk: tile_of_block's, over the pieces of a row.
__global__ __launch_bounds__(kThreads) void probe_update(float *__restrict__ x, const float *__restrict__ g, int64_t d,
                                                         int pieces, int chunk)
{
    const int t = tile_of_block(blockIdx.x, chunk);
    if (t >= pieces) return;
    const int64_t row = (int64_t)blockIdx.y * d;
    const int64_t j0 = (int64_t)t * kTile + 4 * threadIdx.x;
    float4 a[4], b[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + 4 * kThreads * r;
        if (j < d) {
            a[r] = stream_load4(g + row + j);
            b[r] = stream_load4(x + row + j);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = j0 + 4 * kThreads * r;
        if (j < d) st4_stream(x + row + j, make_float4(fadd(a[r].x, b[r].x), fadd(a[r].y, b[r].y), fadd(a[r].z, b[r].z),
                                                       fadd(a[r].w, b[r].w)));
    }
}

}  // namespace cams
