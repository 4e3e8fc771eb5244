// fp32 GEMM on the bf16 matrix cores: every operand split into three bf16 parts, the gather of the selected
// columns inside the tile loads.  Included by cgrad.hip only.
#pragma once
#include "gemm_f32.hpp"

namespace grass {
namespace {

// The fp32 matrix instruction does 256 flop per clock and compute unit, the bf16 one 4096.  A value is
// the exact sum of three bf16 parts (24 significant bits as 8 + 8 + 8, each the nearest bf16 of what the
// ones before leave), so a product of two values is nine exact products of parts; the three least, together
// up to 2^-24 of it (2^-28 is typical), are left out, and six bf16 instructions of 16 tokens stand for eight fp32
// ones of two.  From 8 tokens on the error against 64 bits is smaller than with the fp32 instruction (drawn layers:
// 4e-8 - 9e-8 on the first moment against 6e-8 - 2e-7), because sums are rounded once per 16 tokens and part; below,
// where it would be larger, the fp32 instruction is used (f32_kernel()).
// Operands are multiplied by 2^24 before the split and sums by 2^-48 after the last one: the parts of every
// finite value, subnormal ones included, are then multiples of 2^-125, none of them subnormal or lost.  What is
// too large for that, values from 2^104 and sums from 2^80 on, gives a sum that is not finite, as infinities and NaN
// do; a wavefront that has one does its half of the slice again with the fp32 instruction.  That takes longer than
// the first time (the step of 1024 x 1024, r = 256, T = 8192: 44 us, 108 with one infinity in dY; 4096 x 4096,
// r = 1024, T = 2048: 139 and 439), which a step that is lost anyway may.
//
// A workgroup has eight wavefronts in two groups of four; each group multiplies its half of the slice's
// tokens, and their sums meet in LDS, so that two wavefronts per SIMD hide each other's waits without a
// second partial tile.  Per K tile a wavefront fetches one 32-row fragment of each operand straight into
// registers (lane = row, eight consecutive tokens: the instruction's own layout; loads three tiles ahead),
// splits it (5 vector instructions per value) and writes the parts to one of two LDS stages; the four
// wavefronts then read the fragments they multiply.  BM = BN = 128: 64 x 64 per wavefront, K tiles of 16;
// 64: 32 x 32, K tiles of 32 (two accumulators).
//
// What bounds it: instruction issue and the L2 reads of the gather (each column tile reads the
// lines of the selected columns again) in about equal parts, then the start: the kernel is 10 us long
// before the first token counts.  The step of 1024 x 1024, r = 256, T = 8192: 62 -> 41.5 us (product
// 55 -> 35); 1868 x 1864, r = 467,
// T = 7191: 176 -> 109; 472 x 1480, r = 118, T = 7488, dY stored m x T: 56 -> 32.
constexpr int f32_bk(int bm) { return bm == 128 ? 16 : 32; }  // tokens per K tile
// Row strides (in elements) below this keep a lane's byte offset inside a K tile in 32 bits.  (Rows of a dY stored
// m x T may lie anywhere: they are addressed in 64 bits.)
constexpr int64_t kF32MaxStride = int64_t{1} << 24;

constexpr int kF32Threads = 512, kF32LdsBytes = 96 * 1024;
constexpr float kF32Scale = 0x1p24f, kF32Unscale = 0x1p-48f;  // of each operand; of the sums

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
constexpr int kBufferFlags = 0x00020000;  // 32-bit elements, raw

// a, b as bf16 (nearest even), a in the low half
__device__ __forceinline__ bf16x2 bf16_pair(float a, float b) {
    const f32x2_t v = {a, b};
    return __builtin_convertvector(v, bf16x2);
}

// 16 bytes from an address on a 4-byte boundary
struct __attribute__((packed, aligned(4))) F32Chunk { u32x4_t v; };

// A buffer of the whole address range from token t of a matrix on (rows `bytes` apart).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t f32_buffer(const float* base, uint32_t t, uint32_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base) + static_cast<uint64_t>(t) * bytes;
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p));  // known to be uniform
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((static_cast<uint64_t>(hi) << 32) | lo), 0, -16,
                                             kBufferFlags);
}

// Eight values, times kF32Scale, as the sums of three bf16 each.  kLow, kHigh: (-1, 0) and (0, -1).
struct SplitParts { u32x4_t p[3]; };
__device__ __forceinline__ void split_parts(const float (&x)[8], SplitParts& o, bf16x2 kLow, bf16x2 kHigh) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x0 = x[2 * e] * kF32Scale, x1 = x[2 * e + 1] * kF32Scale;
        const bf16x2 hi = bf16_pair(x0, x1);
        const float r0 = __builtin_amdgcn_fdot2_f32_bf16(hi, kLow, x0, false);
        const float r1 = __builtin_amdgcn_fdot2_f32_bf16(hi, kHigh, x1, false);
        const bf16x2 mid = bf16_pair(r0, r1);
        const float s0 = __builtin_amdgcn_fdot2_f32_bf16(mid, kLow, r0, false);
        const float s1 = __builtin_amdgcn_fdot2_f32_bf16(mid, kHigh, r1, false);
        o.p[0][e] = __builtin_bit_cast(uint32_t, hi);
        o.p[1][e] = __builtin_bit_cast(uint32_t, mid);
        o.p[2][e] = __builtin_bit_cast(uint32_t, bf16_pair(s0, s1));
    }
}

template <int BM, bool kMxT>
__global__ __launch_bounds__(kF32Threads, 2) void tn_gemm_f32_split_kernel(F32Args g) {
    constexpr int BN = BM, F = BM / 64, kFrags = BM / 32;   // F x F fragments of 32 x 32 per wavefront
    constexpr int K16 = f32_bk(BM) / 16, BK = 16 * K16;
    constexpr int kUnit = 512;                              // elements of one part of one fragment
    constexpr int kStage = 2 * kFrags * K16 * 3 * kUnit;
    static_assert(2 * 2 * kStage * 2 == kF32LdsBytes, "two stages for each half of the slice");
    extern __shared__ __attribute__((aligned(16))) uint16_t f32_lds[];

    // consecutive items share a K slice; XCD x receives a contiguous run of items
    // (fewer than 2^31 items; everything derived from the item number is the same for the whole
    // workgroup and is kept in scalar registers)
    const int tiles = g.tiles_m * g.tiles_n, items = tiles * g.splits;
    const int chunk_items = (items + kNumXcd - 1) / kNumXcd;
    const int item = static_cast<int>(blockIdx.x % kNumXcd) * chunk_items + static_cast<int>(blockIdx.x / kNumXcd);
    if (item >= items) return;
    const int split = __builtin_amdgcn_readfirstlane(item / tiles);
    const int tile = __builtin_amdgcn_readfirstlane(item % tiles);
    const int tm = __builtin_amdgcn_readfirstlane(tile % g.tiles_m);
    const int64_t n0 = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(tile / g.tiles_m)) * BN;
    int si = 0;
#pragma unroll
    for (int i = 1; i < GRASS_MAX_GROUP; ++i)
        if (i < g.count && tm >= g.set[i].tile0) si = i;
    const F32Set sg = g.set[si];  // a copy: nothing of the argument block is read inside the loop
    const int64_t row0 = static_cast<int64_t>(tm - sg.tile0) * BM;
    const int T = static_cast<int>(g.T);  // < 2^31
    const int64_t ktiles = (static_cast<int64_t>(T) + BK - 1) / BK;
    const int64_t kt_begin = static_cast<int64_t>(split) * g.ktiles_per_split;
    int64_t kt_end = kt_begin + g.ktiles_per_split;
    if (kt_end > ktiles) kt_end = ktiles;
    const int all = kt_end > kt_begin ? static_cast<int>(kt_end - kt_begin) : 0;

    const int tid = threadIdx.x, lane = tid & 63;
    const int group = __builtin_amdgcn_readfirstlane(tid >> 8), wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
    // this group's half of the slice: `turns` tiles, or one less in the first group (a ragged last tile
    // is then always a tile of the last turn)
    const int turns = __builtin_amdgcn_readfirstlane((all + 1) / 2);
    const int ntiles = group ? turns : all - turns;
    const int t_begin = __builtin_amdgcn_readfirstlane(static_cast<int>((kt_begin + group * (all - turns)) * BK));
    const int t_end = __builtin_amdgcn_readfirstlane(t_begin + ntiles * BK < T ? t_begin + ntiles * BK : T);
    uint16_t* const stages = f32_lds + group * 2 * kStage;
    const int half = lane >> 5, l32 = lane & 31;

    // ---- global -> registers.  This wavefront fetches one fragment of A and one of B per tile: lane =
    // row l32 of the fragment, eight consecutive tokens from krow on.  Rows and columns past the edges
    // are redirected to the first one of the set / matrix (they feed outputs nobody reads).  Past the
    // last whole tile that one is fetched again, unused, so that every trip of the loop issues the same
    // loads (the compiler then waits for the oldest alone).
    const int own_f = K16 == 1 ? wave : wave >> 1, own_s = K16 == 1 ? 0 : wave & 1;
    const int krow = own_s * 16 + half * 8;
    const int64_t ja = row0 + own_f * 32 + l32 < sg.rows ? row0 + own_f * 32 + l32 : 0;
    const int64_t colA = sg.idx ? sg.idx[ja] : ja;
    const int64_t colB = n0 + own_f * 32 + l32 < g.n ? n0 + own_f * 32 + l32 : 0;
    const uint32_t offA = static_cast<uint32_t>((krow * sg.ldy + colA) * 4);  // T x m
    const float* const rowA = sg.dY + colA * sg.ldy + krow;                   // m x T
    const uint32_t offB = static_cast<uint32_t>((krow * g.ldx + colB) * 4);
    struct Raw { float a[8], b[8]; };
    const uint32_t bytesA = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(sg.ldy * 4));
    const uint32_t bytesB = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(g.ldx * 4));
    const int t_whole = __builtin_amdgcn_readfirstlane(
        ntiles > 0 ? t_begin + (t_end - t_begin) / BK * BK - BK : t_begin - BK);  // last whole tile
    auto load = [&](Raw& r, int i) {
        const int at = t_begin + i * BK;
        const uint32_t t0 = __builtin_amdgcn_readfirstlane(at < t_whole ? at : t_whole);
        const auto rb = f32_buffer(g.X, t0, bytesB);
        if (kMxT) {
            const F32Chunk* const src = reinterpret_cast<const F32Chunk*>(rowA + t0);
            const u32x4_t lo = src[0].v, hi = src[1].v;
#pragma unroll
            for (int e = 0; e < 4; ++e) { r.a[e] = __uint_as_float(lo[e]); r.a[4 + e] = __uint_as_float(hi[e]); }
        } else {
            const auto ra = f32_buffer(sg.dY, t0, bytesA);
#pragma unroll
            for (int e = 0; e < 8; ++e) r.a[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, offA, e * bytesA, 0));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) r.b[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, offB, e * bytesB, 0));
    };
    // the ragged last tile, by itself: tokens past T count as 0 (the last token is fetched in their place, so that
    // no load waits for the one before it)
    auto load_ragged = [&](Raw& r, int i) {
        const int t0 = t_begin + i * BK + krow;
        if (t_begin + (i + 1) * BK <= t_end) return;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t t = t0 + e < t_end ? t0 + e : t_end - 1;
            r.a[e] = sg.dY[kMxT ? colA * sg.ldy + t : t * sg.ldy + colA];
            r.b[e] = g.X[t * g.ldx + colB];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (t0 + e >= t_end) r.a[e] = r.b[e] = 0.f;
        }
    };

    // ---- registers -> LDS, split.
    // (-1, 0) and (0, -1) in bf16, kept in registers: an inline -1.0 is not the first to the instruction
    uint32_t low_bits = 0x0000BF80u, high_bits = 0xBF800000u;
    asm("" : "+s"(low_bits), "+s"(high_bits));
    const bf16x2 kLow = __builtin_bit_cast(bf16x2, low_bits), kHigh = __builtin_bit_cast(bf16x2, high_bits);
    auto split8 = [&](const float (&x)[8], uint16_t* dst) {
        SplitParts o;
        split_parts(x, o, kLow, kHigh);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4_t*>(dst + q * kUnit) = o.p[q];
    };
    auto unit = [&](int stage, int operand, int f, int s) {  // `stage`: 0 or kStage
        return stages + stage + ((operand * kFrags + f) * K16 + s) * 3 * kUnit + lane * 8;
    };
    auto split_tile = [&](Raw& r, int stage) {
        split8(r.a, unit(stage, 0, own_f, own_s));
        split8(r.b, unit(stage, 1, own_f, own_s));
    };

    const int wr = wave & 1, wc = wave >> 1;
    f32x16 acc[K16][F][F];
    auto clear = [&]() {
#pragma unroll
        for (int s = 0; s < K16; ++s)
#pragma unroll
            for (int a = 0; a < F; ++a)
#pragma unroll
                for (int b = 0; b < F; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[s][a][b][v] = 0.f;
    };
    clear();
    auto multiply = [&](int stage) {
        bf16x8 fa[K16][F][3], fb[K16][F][3];
#pragma unroll
        for (int s = 0; s < K16; ++s)
#pragma unroll
            for (int p = 2; p >= 0; --p)
#pragma unroll
                for (int a = 0; a < F; ++a) {
                    fa[s][a][p] = *reinterpret_cast<const bf16x8*>(unit(stage, 0, wr * F + a, s) + p * kUnit);
                    fb[s][a][p] = *reinterpret_cast<const bf16x8*>(unit(stage, 1, wc * F + a, s) + p * kUnit);
                }
        __builtin_amdgcn_sched_barrier(0);
        constexpr int kPa[6] = {2, 0, 1, 1, 0, 0}, kPb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int s = 0; s < K16; ++s)
#pragma unroll
                for (int a = 0; a < F; ++a)
#pragma unroll
                    for (int b = 0; b < F; ++b)
                        acc[s][a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][a][kPa[q]], fb[s][b][kPb[q]],
                                                                              acc[s][a][b], 0, 0, 0);
    };
    auto fence = [&]() {  // own LDS accesses done, then everybody's
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // Tile i is multiplied from LDS stage i % 2 while tile i + 1 is split into the other one and three
    // more are in flight.  Both groups take the same number of turns (the barrier is the workgroup's).
    if (turns > 0) {
        Raw R0 = {}, R1 = {}, R2 = {};
        if (t_whole >= t_begin) {
            load(R0, 0);
            load(R1, 1);
            load(R2, 2);
        } else if (ntiles > 0) {
            load_ragged(R0, 0);
        }
        split_tile(R0, 0);
        if (t_whole >= t_begin) load(R0, 3);
        int i = 0, stage = 0;
        auto step = [&](Raw& r, int ahead) {  // r holds tile i + 1 and receives tile `ahead`
            fence();
            multiply(stage);
            stage = kStage - stage;
            split_tile(r, stage);
            load(r, ahead);
        };
        for (; i + 4 < turns; i += 3) {
            step(R1, i + 4);
            step(R2, i + 5);
            step(R0, i + 6);
        }
        // one to four tiles are left: tile i in LDS, the others in R1, R2, R0
        auto last = [&](Raw& r) {
            fence();
            multiply(stage);
            if (++i == turns) return false;
            stage = kStage - stage;
            if (i < ntiles) load_ragged(r, i);
            else r = Raw{};
            split_tile(r, stage);
            return true;
        };
        if (last(R1) && last(R2) && last(R0)) last(R1);
    }
    if (K16 == 2) {
#pragma unroll
        for (int a = 0; a < F; ++a)
#pragma unroll
            for (int b = 0; b < F; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][a][b][v] += acc[K16 - 1][a][b][v];
    }

    // A sum that is not finite (an input that is not, or that is too large for its parts): this wavefront's block
    // again, with the fp32 instruction.
    float finite = 0.f;  // stays 0
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
        for (int b = 0; b < F; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) finite = __builtin_fmaf(acc[0][a][b][v], 0.f, finite);
    if (!__any(finite != 0.f)) {
#pragma unroll
        for (int a = 0; a < F; ++a)
#pragma unroll
            for (int b = 0; b < F; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][a][b][v] *= kF32Unscale;
    } else {
        clear();
        const int64_t strideA = kMxT ? 1 : sg.ldy;
        const float *pa[F], *pb[F];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const int64_t j = row0 + wr * (BM / 2) + f * 32 + l32, c = n0 + wc * (BN / 2) + f * 32 + l32;
            const int64_t src = sg.idx ? sg.idx[j < sg.rows ? j : 0] : (j < sg.rows ? j : 0);
            pa[f] = sg.dY + (kMxT ? src * sg.ldy : src);
            pb[f] = g.X + (c < g.n ? c : 0);
        }
        for (int t0 = t_begin; ntiles > 0 && t0 < t_end; t0 += 16) {
            float fa[8][F], fb[8][F];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool in = t_end - t0 > 2 * k + half;
                const int64_t t = in ? t0 + 2 * k + half : t_end - 1;
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const float a = pa[f][t * strideA], b = pb[f][t * g.ldx];
                    fa[k][f] = in ? a : 0.f;
                    fb[k][f] = in ? b : 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int a = 0; a < F; ++a)
#pragma unroll
                    for (int b = 0; b < F; ++b)
                        acc[0][a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[k][a], fb[k][b], acc[0][a][b], 0, 0, 0);
        }
    }

    // The two groups' sums meet: each gives half of its accumulators to the other through LDS and stores
    // the half it keeps.  Element e = (a F + b) 16 + v of lane l is C[8*(v/4) + 4*(l/32) + v%4][l%32] of
    // fragment (a, b).
    constexpr int kKeep = F * F * 8;
    float* const lds = reinterpret_cast<float*>(f32_lds);
    auto element = [&](int e) -> float { return acc[0][e / (16 * F)][e / 16 % F][e % 16]; };
    __syncthreads();
    auto give = [&](int first) {
#pragma unroll
        for (int q = 0; q < kKeep / 4; ++q)
            *reinterpret_cast<float4*>(lds + ((group * (kKeep / 4) + q) * 256 + (tid & 255)) * 4) =
                make_float4(element(first + 4 * q), element(first + 4 * q + 1), element(first + 4 * q + 2), element(first + 4 * q + 3));
    };
    const int64_t left = sg.rows - row0 - wr * (BM / 2);  // rows of this wavefront's block that exist
    auto finish = [&](int first) {
        float sum[kKeep];
#pragma unroll
        for (int q = 0; q < kKeep / 4; ++q) {
            const float4 o = *reinterpret_cast<const float4*>(lds + (((1 - group) * (kKeep / 4) + q) * 256 + (tid & 255)) * 4);
            sum[4 * q] = element(first + 4 * q) + o.x;
            sum[4 * q + 1] = element(first + 4 * q + 1) + o.y;
            sum[4 * q + 2] = element(first + 4 * q + 2) + o.z;
            sum[4 * q + 3] = element(first + 4 * q + 3) + o.w;
        }
        // elements that lie in the same row, F of them 16 apart, belong to the fragments b
        constexpr int kRows = F == 1 ? kKeep : 16;
        if (g.P) {
            float* P = g.P + (static_cast<int64_t>(split) * g.Mp + sg.off + row0 + wr * (BM / 2)) * g.Np + n0 +
                       wc * (BN / 2) + l32;
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const int v = (first + k) % 16, row = first / (16 * F) * 32 + 8 * (v / 4) + 4 * half + (v % 4);
                if (row >= left) continue;
#pragma unroll
                for (int b = 0; b < F; ++b) P[row * g.Np + b * 32] = sum[b * 16 + k];
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int v = (first + k) % 16, row_in = first / (16 * F) * 32 + 8 * (v / 4) + 4 * half + (v % 4);
            if (row_in >= left) continue;
            const int64_t row = row0 + wr * (BM / 2) + row_in;
            const float s = sg.rho ? sg.rho[row] : 1.0f;
#pragma unroll
            for (int b = 0; b < F; ++b) {
                const int64_t col = n0 + wc * (BN / 2) + b * 32 + l32;
                if (col >= g.n) continue;
                if (g.c_bf16) store_from_f32(static_cast<uint16_t*>(sg.C) + row * sg.ldc + col, s * sum[b * 16 + k]);
                else store_from_f32(static_cast<float*>(sg.C) + row * sg.ldc + col, s * sum[b * 16 + k]);
            }
        }
    };
    if (group == 0) {
        give(kKeep);
        __syncthreads();
        finish(0);
    } else {
        give(0);
        __syncthreads();
        finish(kKeep);
    }
}

}  // namespace
}  // namespace grass
