// First layer's FFN input of the bf16 kernels: xn = x * g (or x without a norm) in bf16, plus the row's sums of
// squares for the RMSNorm factor.  Also the identity index lists with which the dense reference runs the
// sparse kernels, and the launch that runs the mask compaction beside the prologue (the calls that take masks).
//
// The action expert normalizes each FFN input (the layer is x + FFN(RMSNorm(x)) with RMSNorm(x) =
// x / sqrt(mean(x^2) + eps) * g).  The per-token factor is applied by the gate/up kernel after its matrix-core
// products, so xn itself stays unscaled.  One wave per (token row, block of 256 columns), each lane a float4:
// the row's sum of squares is kept as one partial per column block (lane butterfly, fixed order), which the
// gate/up kernel adds in block order.
#include <algorithm>

#include "rm_units.h"

namespace {

constexpr int kThreads = 64;

__global__ __launch_bounds__(kThreads) void prologue_kernel(const float *__restrict__ x,
                                                            const float *__restrict__ g, int d, int nblk,
                                                            uint16_t *__restrict__ xn, float *__restrict__ ssq) {
    rm_units::prologue_unit(x, g, d, nblk, xn, ssq, blockIdx.x, threadIdx.x);
}

// Compaction and prologue in one launch (they are independent): workgroups [0, n_compact) each compact one
// (mask, segment) unit; each later workgroup runs the prologue of four (row, column block) units, one per wave.
__global__ __launch_bounds__(rm_units::kCompactThreads) void compact_prologue_kernel(
    const uint8_t *__restrict__ mask, int d_ff, int nseg, int n_compact, int32_t *__restrict__ idx,
    int32_t *__restrict__ count, const float *__restrict__ x, const float *__restrict__ g, int d, int nblk,
    int units, uint16_t *__restrict__ xn, float *__restrict__ ssq) {
    const int w = static_cast<int>(blockIdx.x);
    if (w < n_compact) {
        const int m = w / nseg;
        rm_units::compact_segment(mask, d_ff, m, w - m * nseg, idx, count);
        return;
    }
    const int unit = (w - n_compact) * (rm_units::kCompactThreads / 64) + static_cast<int>(threadIdx.x >> 6);
    if (unit < units) rm_units::prologue_unit(x, g, d, nblk, xn, ssq, unit, threadIdx.x & 63);
}

// The lists 0 .. d_ff-1 and counts d_ff of B samples, by `groups` workgroups of 256 threads, this one the w-th.
__device__ __forceinline__ void identity_lists(int32_t *idx, int32_t *count, int d_ff, int B, int w, int groups) {
    const size_t n = static_cast<size_t>(B) * d_ff;
    const size_t step = static_cast<size_t>(groups) * 256;
    for (size_t i = static_cast<size_t>(w) * 256 + threadIdx.x; i < n; i += step) idx[i] = static_cast<int32_t>(i % d_ff);
    for (int b = threadIdx.x; w == 0 && b < B; b += 256) count[b] = d_ff;
}

__global__ __launch_bounds__(256) void identity_lists_kernel(int32_t *idx, int32_t *count, int d_ff, int B) {
    identity_lists(idx, count, d_ff, B, blockIdx.x, gridDim.x);
}

// The identity lists and the prologue in one launch (they are independent), as the compaction and the prologue:
// workgroups [0, n_lists) write the lists, each later one runs four prologue units.
__global__ __launch_bounds__(256) void identity_prologue_kernel(int32_t *idx, int32_t *count, int d_ff, int B,
                                                                int n_lists, const float *__restrict__ x,
                                                                const float *__restrict__ g, int d, int nblk, int units,
                                                                uint16_t *__restrict__ xn, float *__restrict__ ssq) {
    const int w = static_cast<int>(blockIdx.x);
    if (w < n_lists) {
        identity_lists(idx, count, d_ff, B, w, n_lists);
        return;
    }
    const int unit = (w - n_lists) * 4 + static_cast<int>(threadIdx.x >> 6);
    if (unit < units) rm_units::prologue_unit(x, g, d, nblk, xn, ssq, unit, threadIdx.x & 63);
}

}  // namespace

namespace rm {

hipError_t launch_identity_lists(const Plan &p, void *ws, hipStream_t st) {
    char *base = static_cast<char *>(ws);
    int32_t *idx = reinterpret_cast<int32_t *>(base + p.off_ident);
    int32_t *count = reinterpret_cast<int32_t *>(base + p.off_ident_count);
    const size_t n = static_cast<size_t>(p.B) * p.d_ff;
    const int blocks = static_cast<int>(std::min<size_t>((n + 255) / 256, 1024));
    hipLaunchKernelGGL(identity_lists_kernel, dim3(blocks), dim3(256), 0, st, idx, count, p.d_ff, p.B);
    return hipGetLastError();
}

hipError_t launch_identity_prologue(const Plan &p, const float *x, const float *norm_g, void *ws, hipStream_t st) {
    char *base = static_cast<char *>(ws);
    int32_t *idx = reinterpret_cast<int32_t *>(base + p.off_ident);
    int32_t *count = reinterpret_cast<int32_t *>(base + p.off_ident_count);
    const size_t n = static_cast<size_t>(p.B) * p.d_ff;
    const int n_lists = static_cast<int>(std::min<size_t>((n + 255) / 256, 1024));
    const int nblk = (p.d + kRowBlock - 1) / kRowBlock;
    const int units = p.B * p.T * nblk;
    // A grid of 2^32 threads or more wraps without an error: where the lists' workgroups do not fit beside the
    // prologue's, two launches.
    if ((n_lists + (units + 3LL) / 4) * 256 > 0xffffffffLL) {
        const hipError_t e = launch_identity_lists(p, ws, st);
        return e != hipSuccess ? e : launch_prologue(p, x, norm_g, ws, st);
    }
    hipLaunchKernelGGL(identity_prologue_kernel, dim3(n_lists + (units + 3) / 4), dim3(256), 0, st, idx, count, p.d_ff,
                       p.B, n_lists, x, norm_g, p.d, nblk, units, reinterpret_cast<uint16_t *>(base + p.off_xn),
                       reinterpret_cast<float *>(base + p.off_ssq));
    return hipGetLastError();
}

hipError_t launch_compact_prologue(const Plan &p, const uint8_t *mask, int n_masks, int32_t *idx, int32_t *count,
                                   const float *x, const float *norm_g, void *ws, hipStream_t st) {
    char *base = static_cast<char *>(ws);
    uint16_t *xn = reinterpret_cast<uint16_t *>(base + p.off_xn);
    float *ssq = reinterpret_cast<float *>(base + p.off_ssq);
    const int nblk = (p.d + kRowBlock - 1) / kRowBlock;
    const int nseg = (p.d_ff + rm_units::kSeg - 1) / rm_units::kSeg;
    const int n_compact = nseg * n_masks;
    const int units = p.B * p.T * nblk;
    const int per = rm_units::kCompactThreads / 64;
    const dim3 grid(n_compact + (units + per - 1) / per);
    const dim3 block(rm_units::kCompactThreads);
    hipLaunchKernelGGL(compact_prologue_kernel, grid, block, 0, st, mask, p.d_ff, nseg, n_compact, idx,
                       count, x, norm_g, p.d, nblk, units, xn, ssq);
    return hipGetLastError();
}

hipError_t launch_prologue(const Plan &p, const float *x, const float *norm_g, void *ws, hipStream_t st) {
    char *base = static_cast<char *>(ws);
    uint16_t *xn = reinterpret_cast<uint16_t *>(base + p.off_xn);
    float *ssq = reinterpret_cast<float *>(base + p.off_ssq);
    const int nblk = (p.d + kRowBlock - 1) / kRowBlock;
    const dim3 grid(p.B * p.T * nblk);
    hipLaunchKernelGGL(prologue_kernel, grid, dim3(kThreads), 0, st, x, norm_g, p.d, nblk, xn, ssq);
    return hipGetLastError();
}

}  // namespace rm
