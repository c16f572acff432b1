// Vanilla distributed AMSGrad without compression (Section 3): gbar = (1/n) sum_i g_i in ascending
// worker order, then the AMSGrad update.
// Traffic: 4 B (2 B for 16-bit gradients) per (worker, coordinate) + 32 B per coordinate; HBM-bound.
//
// One workgroup per quarter of a tile, one float4 of coordinates per thread, the workers' rows one after the
// other: few registers, so the compute units are full of wavefronts and those hide each other's loads, and four
// times as many workgroups, so a short vector fills the chip.  Against four float4 per thread with the loads of
// four workers in flight (three sets of buffers in turn, us): n = 16, d = 11.2 M bf16 172 -> 125, fp32 188 -> 182;
// n = 32, d = 25.6 M bf16 529 -> 425, fp32 734 -> 725; n = 8, d = 110 M bf16 912 -> 888, fp32 1.25 -> 1.23 ms;
// n = 16, d = 1.2 M bf16 49 -> 22, fp32 33 -> 24.  Batches of 2 to 16 rows in flight lose up to 10 % on fp32 (16 bits:
// see plain_rows_ahead); eight 16-bit gradients per lane (16-byte loads) take twice as long, because the state is then
// written in half lines.
#pragma once
#include "device_utils.h"

namespace cams {

constexpr int kPlainCoords = 4 * kThreads;   // coordinates per workgroup: a quarter of a tile

// acc += the coordinates j .. j + 3 of the n rows, in ascending order, kAhead rows loaded at a time (see plain_rows_ahead).
template <bool kInside, int kAhead, typename G>
__device__ __forceinline__ void sum_rows(float4 &acc, const G *__restrict__ row, int64_t j, int64_t d, int n)
{
    auto add = [&](const float4 &x) {
        acc.x = fadd(acc.x, x.x);
        acc.y = fadd(acc.y, x.y);
        acc.z = fadd(acc.z, x.z);
        acc.w = fadd(acc.w, x.w);
    };
    int i = 0;
#pragma unroll 1
    for (; i + kAhead <= n; i += kAhead, row += kAhead * d) {
        GradRaw<G> x[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) x[u] = load_raw4<kInside>(row + u * d, j, d);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) add(widen4(x[u]));
    }
#pragma unroll 1
    for (; i < n; ++i, row += d) add(widen4(load_raw4<kInside>(row, j, d)));
}

template <typename G, bool kStreamState, int kAhead>   // G: float, uint16_t (bfloat16 bits) or f16bits
__global__ __launch_bounds__(kThreads) void plain_update(const G *__restrict__ g, int64_t d, int n,
                                                         float *__restrict__ theta, float *__restrict__ m,
                                                         float *__restrict__ v, float *__restrict__ vhat, AmsParams p, int chunk,
                                                         int n_quarters)
{
    const int t = tile_of_block(blockIdx.x, chunk);
    if (t >= n_quarters) return;
    const int64_t j = (int64_t)t * kPlainCoords + 4 * threadIdx.x;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (((int64_t)t + 1) * kPlainCoords <= d)
        sum_rows<true, kAhead>(acc, g, j, d, n);
    else
        sum_rows<false, kAhead>(acc, g, j, d, n);
    float4 th = ld4_state<kStreamState>(theta + j), mm = ld4_state<kStreamState>(m + j),
           vv = ld4_state<kStreamState>(v + j), vh = ld4_state<kStreamState>(vhat + j);
    // padding coordinates take no gradient (load_raw4 gives 0 past d)
    const float4 gbar = make_float4(fdiv(acc.x, p.n_workers), fdiv(acc.y, p.n_workers), fdiv(acc.z, p.n_workers),
                                    fdiv(acc.w, p.n_workers));
    amsgrad_update4(th, mm, vv, vh, gbar, p);
    st4_state<kStreamState>(theta + j, th);
    st4_state<kStreamState>(m + j, mm);
    st4_state<kStreamState>(v + j, vv);
    st4_state<kStreamState>(vhat + j, vh);
}

}  // namespace cams
