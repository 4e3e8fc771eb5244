// fp32 products over few tokens: 32 x 32 tiles, K divided over the wavefronts of one workgroup, and,
// where a set fits one row tile, the rest of a regular step in the same launch.  Included by cgrad.hip only.
#pragma once
#include "adam.hpp"
#include "gemm_f32_split.hpp"

namespace grass {
namespace {

// What bounds a short product is neither arithmetic nor bandwidth but its start and end: the launch, the
// chain row index -> element -> product, cold instructions, partial tiles and the launch that sums them.
// So a workgroup keeps all of K: its sixteen wavefronts take every sixteenth chunk of 16 tokens, fetch their
// operands straight into registers (lane = row of the fragment, eight tokens each: the layout the
// matrix instruction wants, no LDS and no barrier in the loop), split them as in gemm_f32_split.hpp, and meet
// once in LDS.  Nothing is summed by a second kernel; a set of at most 32 rows lies in one tile, whose
// workgroup then also does Adam and the update of W (runs of equal idx included), with the moments and
// weights fetched before the product.
constexpr int kShortWaves = 16, kShortTile = 32;

// The tail of a regular step, for the fused form.
struct F32StepSet {
    void* M;
    void* V;
    void* W;
    int64_t ldw;
    float* GC;  // or nullptr
    int64_t ldgc;
};
struct F32StepArgs {
    F32StepSet set[GRASS_MAX_GROUP];
    AdamParams adam;
    float alpha;
    int s_bf16, w_bf16;
};

__device__ __forceinline__ float load_either(const void* p, int64_t i, int bf16) {
    return bf16 ? bf16_to_f32(static_cast<const uint16_t*>(p)[i]) : static_cast<const float*>(p)[i];
}
__device__ __forceinline__ void store_either(void* p, int64_t i, int bf16, float v) {
    if (bf16) static_cast<uint16_t*>(p)[i] = f32_to_bf16(v);
    else static_cast<float*>(p)[i] = v;
}

template <bool kMxT, bool kStep>
__global__ __launch_bounds__(kShortWaves * 64) void tn_gemm_f32_short_kernel(F32Args g, F32StepArgs step) {
    constexpr int kOwn = 16 / kShortWaves;  // accumulator elements a wavefront sums and finishes
    __shared__ float share[kShortWaves / 2][16][64];
    __shared__ float u_tile[kShortTile][kShortTile + 1];
    const int tm = static_cast<int>(blockIdx.x) % g.tiles_m, tn = static_cast<int>(blockIdx.x) / g.tiles_m;
    int si = 0;
#pragma unroll
    for (int i = 1; i < GRASS_MAX_GROUP; ++i)
        if (i < g.count && tm >= g.set[i].tile0) si = i;
    const F32Set sg = g.set[si];
    const int64_t row0 = static_cast<int64_t>(tm - sg.tile0) * kShortTile, n0 = static_cast<int64_t>(tn) * kShortTile;
    const int T = static_cast<int>(g.T);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const bool row_ok = row0 + l32 < sg.rows, col_ok = n0 + l32 < g.n;
    const int64_t ja = row_ok ? row0 + l32 : 0, colB = col_ok ? n0 + l32 : 0;
    const int64_t colA = sg.idx ? sg.idx[ja] : ja;

    // ---- the step's own operands, on their way while the product is formed.  This thread finishes
    // elements v = wave * kOwn + k: row 8 (v / 4) + 4 half + v % 4, column l32 of the tile.
    int64_t row[kOwn], at[kOwn];  // compressed row; its element of M and V
    int32_t w_row[kOwn];
    float m[kOwn], v[kOwn], w[kOwn], scale[kOwn];
    bool live[kOwn], leads[kOwn];
    const F32StepSet ss = step.set[si];
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
        const int e = wave * kOwn + k;
        row[k] = row0 + 8 * (e / 4) + 4 * half + (e % 4);
        live[k] = row[k] < sg.rows && col_ok;
        scale[k] = 1.f;
        if (!kStep || !live[k]) continue;
        at[k] = row[k] * g.n + n0 + l32;
        scale[k] = sg.rho[row[k]];
        m[k] = load_either(ss.M, at[k], step.s_bf16);
        v[k] = load_either(ss.V, at[k], step.s_bf16);
        w_row[k] = sg.idx[row[k]];
        leads[k] = row[k] == 0 || sg.idx[row[k] - 1] != w_row[k];
        if (leads[k]) w[k] = load_either(ss.W, w_row[k] * ss.ldw + n0 + l32, step.w_bf16);
    }

    // ---- the product
    const int64_t strideA = kMxT ? 1 : sg.ldy;
    const float* const pa = sg.dY + (kMxT ? colA * sg.ldy : colA);
    const float* const pb = g.X + colB;
    struct Raw { float a[8], b[8]; };
    const int chunks = (T + 15) / 16;
    const uint32_t offA = static_cast<uint32_t>((half * 8 * sg.ldy + colA) * 4);  // T x m
    const uint32_t offB = static_cast<uint32_t>((half * 8 * g.ldx + colB) * 4);
    const uint32_t bytesA = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(sg.ldy * 4));
    const uint32_t bytesB = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(g.ldx * 4));
    const int whole = __builtin_amdgcn_readfirstlane(T / 16);
    auto load = [&](Raw& r, int c) {  // past the last whole chunk: that one again, unused
        const uint32_t t = __builtin_amdgcn_readfirstlane((c < whole ? c : whole - 1) * 16);
        const auto ra = f32_buffer(sg.dY, t, bytesA), rb = f32_buffer(g.X, t, bytesB);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            r.a[e] = kMxT ? pa[t + half * 8 + e] : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, offA, e * bytesA, 0));
            r.b[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, offB, e * bytesB, 0));
        }
    };
    uint32_t low_bits = 0x0000BF80u, high_bits = 0xBF800000u;  // see gemm_f32_split.hpp
    asm("" : "+s"(low_bits), "+s"(high_bits));
    const bf16x2 kLow = __builtin_bit_cast(bf16x2, low_bits), kHigh = __builtin_bit_cast(bf16x2, high_bits);
    f32x16 acc[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.f;
    auto multiply = [&](const Raw& r) {
        SplitParts a, b;
        split_parts(r.a, a, kLow, kHigh);
        split_parts(r.b, b, kLow, kHigh);
        auto product = [&](int i, int j, int k) {
            acc[k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.p[i]), __builtin_bit_cast(bf16x8, b.p[j]), acc[k], 0, 0, 0);
        };
        product(2, 0, 0); product(0, 2, 1); product(1, 1, 0); product(1, 0, 1); product(0, 1, 0); product(0, 0, 1);
    };
    {
        Raw r0, r1;
        if (wave < whole) {
            load(r0, wave);
            for (int c = wave;; c += 2 * kShortWaves) {
                load(r1, c + kShortWaves);
                multiply(r0);
                if (c + kShortWaves >= whole) break;
                load(r0, c + 2 * kShortWaves);
                multiply(r1);
                if (c + 2 * kShortWaves >= whole) break;
            }
        }
        if (T % 16 != 0 && wave == whole % kShortWaves) {  // the last chunk: tokens past T count as 0
            const int first = whole * 16 + half * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) {  // the last token in place of those: no load waits for the one before it
                const int t = first + e < T ? first + e : T - 1;
                r0.a[e] = pa[t * strideA];
                r0.b[e] = pb[t * g.ldx];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (first + e >= T) r0.a[e] = r0.b[e] = 0.f;
            }
            multiply(r0);
        }
    }
    float finite = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        acc[0][e] += acc[1][e];
        finite = __builtin_fmaf(acc[0][e], 0.f, finite);
    }
    if (!__any(finite != 0.f)) {  // see gemm_f32_split.hpp
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[0][e] *= kF32Unscale;
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[0][e] = 0.f;
        for (int c = wave; c < chunks; c += kShortWaves) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool in = T - c * 16 > 2 * k + half;
                const int64_t t = in ? c * 16 + 2 * k + half : T - 1;
                const float a = pa[t * strideA], b = pb[t * g.ldx];
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? a : 0.f, in ? b : 0.f, acc[0], 0, 0, 0);
            }
        }
    }
    // the upper half of the wavefronts hands its sums to the lower one, then all meet
    constexpr int kHalfWaves = kShortWaves / 2;
    if (wave >= kHalfWaves)
#pragma unroll
        for (int e = 0; e < 16; ++e) share[wave - kHalfWaves][e][lane] = acc[0][e];
    __syncthreads();
    if (wave < kHalfWaves)
#pragma unroll
        for (int e = 0; e < 16; ++e) share[wave][e][lane] += acc[0][e];
    __syncthreads();
    float sum[kOwn];
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
        sum[k] = 0.f;
#pragma unroll
        for (int q = 0; q < kHalfWaves; ++q) sum[k] += share[q][wave * kOwn + k][lane];
    }
    if (!kStep) {
#pragma unroll
        for (int k = 0; k < kOwn; ++k) {
            if (!live[k]) continue;
            const int64_t col = n0 + l32;
            if (g.P) {
                g.P[(sg.off + row[k]) * g.Np + col] = sum[k];
            } else {
                const float x = (sg.rho ? sg.rho[row[k]] : 1.f) * sum[k];
                if (g.c_bf16) store_from_f32(static_cast<uint16_t*>(sg.C) + row[k] * sg.ldc + col, x);
                else store_from_f32(static_cast<float*>(sg.C) + row[k] * sg.ldc + col, x);
            }
        }
        return;
    }
    const AdamParams p = resolve(step.adam);
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
        if (!live[k]) continue;
        const float gk = sum[k] * scale[k];
        if (ss.GC) ss.GC[row[k] * ss.ldgc + n0 + l32] = gk;
        u_tile[row[k]][l32] = step.s_bf16 ? adam_elem<uint16_t>(gk, m[k], v[k], p) : adam_elem<float>(gk, m[k], v[k], p);
        store_either(ss.M, at[k], step.s_bf16, m[k]);
        store_either(ss.V, at[k], step.s_bf16, v[k]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
        if (!live[k] || !leads[k]) continue;
        float sum_u = 0.f;
        for (int64_t j = row[k]; j < sg.rows && sg.idx[j] == w_row[k]; ++j) sum_u += sg.rho[j] * u_tile[j][l32];
        w[k] += step.alpha * sum_u;
        store_either(ss.W, w_row[k] * ss.ldw + n0 + l32, step.w_bf16, w[k]);
    }
}

}  // namespace
}  // namespace grass
