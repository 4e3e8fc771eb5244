// Adam's scalars and its update of one element, shared by the kernels that end in it.
#pragma once
#include "common.hpp"

namespace grass {
namespace {

struct AdamParams {
    float b1, one_minus_b1, b2, one_minus_b2;
    float inv_c1, inv_c2;  // reciprocals of the bias corrections 1 - beta^t
    float lr, eps;
    // When set: device array {lr, inv_c1, inv_c2} that replaces the three values above, so that
    // a captured launch can be replayed for later steps (the caller rewrites the array).
    const float* step_scalars;
};

// The values of this step: from the launch arguments, or from device memory.
__device__ __forceinline__ AdamParams resolve(AdamParams p) {
    if (p.step_scalars) {
        p.lr = p.step_scalars[0];
        p.inv_c1 = p.step_scalars[1];
        p.inv_c2 = p.step_scalars[2];
    }
    return p;
}

// What a moment becomes when it is stored: itself in fp32, the nearest bf16 value otherwise.
template <typename ST>
__device__ __forceinline__ float as_stored(float x);
template <>
__device__ __forceinline__ float as_stored<float>(float x) { return x; }
template <>
__device__ __forceinline__ float as_stored<uint16_t>(float x) { return bf16_to_f32(f32_to_bf16(x)); }

// adam.update of Appendix A for one element; returns U.  With bf16 moments the update is
// computed from the values that are stored, so it is a function of the saved state.
template <typename ST>
__device__ __forceinline__ float adam_elem(float g, float& m, float& v, const AdamParams& p) {
    m = as_stored<ST>(p.b1 * m + p.one_minus_b1 * g);
    v = as_stored<ST>(p.b2 * v + p.one_minus_b2 * g * g);
    const float ms = m * p.inv_c1;
    const float vs = v * p.inv_c2;
    // hardware square root and reciprocal (about 1 ulp each): the kernel is otherwise bound by
    // memory and the correctly rounded sequences would make its arithmetic show
    return -p.lr * ms * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(vs) + p.eps);
}

AdamParams make_params(float lr, float b1, float b2, float eps, int64_t t,
                       const float* step_scalars) {
    AdamParams p;
    p.step_scalars = step_scalars;
    if (t < 1) t = 1;  // unused when step_scalars is set
    p.b1 = b1;
    p.one_minus_b1 = 1.0f - b1;
    p.b2 = b2;
    p.one_minus_b2 = 1.0f - b2;
    p.inv_c1 = static_cast<float>(1.0 / (1.0 - pow(static_cast<double>(b1), static_cast<double>(t))));
    p.inv_c2 = static_cast<float>(1.0 / (1.0 - pow(static_cast<double>(b2), static_cast<double>(t))));
    p.lr = lr;
    p.eps = eps;
    return p;
}

}  // namespace
}  // namespace grass
