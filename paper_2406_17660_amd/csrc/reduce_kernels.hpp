// Split-K and row-statistic reductions.
// Included by cgrad.hip only (device code shares one translation unit with its launchers).
#pragma once
#include "common.hpp"
#include "gemm_common.hpp"

namespace grass {
namespace {

// sumsq[k] = sum over the column slots of rowpart[slot][k], in slot order (deterministic)
__global__ __launch_bounds__(256) void rowpart_reduce_kernel(const float* __restrict__ part, int slots,
                                                             int64_t Mp, int64_t m,
                                                             float* __restrict__ sumsq) {
    const int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (k >= m) return;
    float s = 0.f;
    for (int i = 0; i < slots; ++i) s += part[static_cast<int64_t>(i) * Mp + k];
    sumsq[k] = s;
}

// out[j, i] = scale_j * sum_s P[s][j][i]   (fixed summation order: deterministic)
// A thread owns four columns, 256 apart, so that four loads per slice are in flight while rows of
// out may start anywhere
// (5461 x 2048 from four slices: 62 us with one column per thread, 57 us so).
constexpr int kReduceCols = 4;
template <typename OT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ P, int splits,
                                                            int64_t Mp, int64_t Np, int64_t rows,
                                                            int64_t cols,
                                                            const float* __restrict__ scale,
                                                            OT* __restrict__ out, int64_t ldo) {
    const int64_t j = blockIdx.y;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * 256 * kReduceCols, i = first + threadIdx.x;
    if (i >= cols) return;
    float s[kReduceCols] = {0.f, 0.f, 0.f, 0.f};
    const float* src = P + j * Np + first;
    const int64_t step = Mp * Np;
    uint32_t lane[kReduceCols];  // past the edge: the thread's first column again
#pragma unroll
    for (int u = 0; u < kReduceCols; ++u) lane[u] = (threadIdx.x + (i + u * 256 < cols ? u * 256 : 0)) * 4;
    add_columns(src, lane, step, splits, s);
    const float sc = scale ? scale[j] : 1.0f;
#pragma unroll
    for (int u = 0; u < kReduceCols; ++u)
        if (i + u * 256 < cols) store_from_f32(out + j * ldo + i + u * 256, s[u] * sc);
}

// The same sum for many slices (short, wide problems split K dozens of times): one workgroup
// per output row and 256 columns; each of its four wavefronts adds a contiguous quarter of the
// slices, four columns per lane, and the four partial sums are added in wavefront order.  The
// order is fixed, so the result does not change from run to run.
template <typename OT>
__global__ __launch_bounds__(256) void splitk_reduce_many_kernel(
    const float* __restrict__ P, int splits, int64_t Mp, int64_t Np, int64_t rows, int64_t cols,
    const float* __restrict__ scale, OT* __restrict__ out, int64_t ldo) {
    __shared__ float4 part[4][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t j = blockIdx.y;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + lane * 4;  // < Np: Np % 128 == 0
    const int per = (splits + 3) / 4;
    const int k0 = w * per, k1 = k0 + per < splits ? k0 + per : splits;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (i < Np)
        add_slices(P + (static_cast<int64_t>(k0) * Mp + j) * Np + static_cast<int64_t>(blockIdx.x) * 256, lane * 16, Mp * Np, k1 - k0, s);
    part[w][lane] = make_float4(s[0], s[1], s[2], s[3]);
    __syncthreads();
    if (w != 0 || i >= cols) return;
    float r[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = part[q][lane];
        r[0] += v.x; r[1] += v.y; r[2] += v.z; r[3] += v.w;
    }
    const float sc = scale ? scale[j] : 1.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (i + e < cols) store_from_f32(out + j * ldo + i + e, r[e] * sc);
}

}  // namespace
}  // namespace grass
