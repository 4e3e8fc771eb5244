// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products, fp32 accumulation) with
// the gather of the selected columns inside the tile loads.  Included by cgrad.hip only.
#pragma once
#include "gemm_large.hpp"  // load-to-LDS helpers, wait_vmcnt

namespace grass {
namespace {

// What bounds it: the matrix instruction itself (256 flop per clock and compute unit, 157 TFLOP/s
// on the chip).  An operand of it is one float per lane and step of two k, read from a t-major
// LDS tile as it lies in memory: no transposition, and 64 clocks of matrix pipe per LDS read
// pair, so LDS bandwidth does not matter and the tile can be small.  What does matter is having
// enough workgroups: the outputs of fp32 layers are small (r x n of a few hundred by a thousand)
// and K is long, so K is split until the machine is full, and each workgroup keeps three K tiles
// of 16 tokens in flight through a four-stage LDS ring (load-to-LDS, waits placed by hand).
// The left operand is gathered by the loads: one lane fetches one selected column (4 bytes;
// 64 selected columns lie in a few cache lines of a row of dY, and each of the n / BN column tiles
// reads them once more from L2), which costs less than a packing pass would.  dY stored m x T is
// read the same way, lane = row: 16 consecutive t share a cache line through L1.
//
// Four wavefronts of 32 x 32 on a 64 x 64 tile.  Small products only: it starts 3 - 4 us sooner than the
// kernel with split operands (gemm_f32_split.hpp), which is up to 1.75 times as fast on large ones; the
// line between them is in f32_kernel().
constexpr int kF32Tile = 64, kF32BK = 16, kF32Stages = 4;

struct F32Set {
    const float* dY;
    int64_t ldy;
    const int32_t* idx;  // `rows` columns of dY, or nullptr: column j itself
    const float* rho;    // scales of the direct output (nullptr: 1)
    void* C;             // direct output (used when P is nullptr)
    int64_t ldc;
    int64_t rows;
    int64_t off;         // first row of this set in the partial tiles
    int tile0;           // row tiles of the sets before this one
};
struct F32Args {
    F32Set set[GRASS_MAX_GROUP];
    int count;
    const float* X;
    int64_t ldx, n, T;
    float* P;            // partial tiles [splits][Mp][Np], or nullptr: store scale * sum to C
    int64_t Mp, Np;
    int mxt;             // dY stored m x T
    int c_bf16;          // direct output in bf16
    int tiles_m, tiles_n, splits, ktiles_per_split;
};

// 4 bytes per lane: lane i of the wavefront writes LDS bytes [lds_base + 4*i, +4).
__device__ __forceinline__ void load4_to_lds(const void* lane_addr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dword %0, off"
                 :
                 : "v"(lane_addr), "s"(lds_base)
                 : "memory", "m0");
}

// kVecA: dense left operand (no idx, T x m), 16-byte loads; kVecB: 16-byte loads of X.
template <bool kVecA, bool kVecB>
__global__ __launch_bounds__(256, 4) void tn_gemm_f32_mfma_kernel(F32Args g) {
    constexpr int BM = kF32Tile, BN = kF32Tile, BK = kF32BK, F = BM / 64;  // F x F fragments of 32 x 32 per wavefront
    constexpr int kOperand = BK * BM;                 // floats of one operand of one stage
    constexpr int kLoadsA = kVecA ? F : 4 * F, kLoadsB = kVecB ? F : 4 * F, kLoads = kLoadsA + kLoadsB;
    __shared__ __attribute__((aligned(1024))) float ring[kF32Stages * 2 * kOperand];

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
    const int ntiles = kt_end > kt_begin ? static_cast<int>(kt_end - kt_begin) : 0;
    const int t_begin = static_cast<int>(kt_begin * BK);  // used when ntiles > 0: then below T

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- global -> LDS.  Rows and columns past the edges are redirected to the first one of the
    // set / matrix (they feed outputs nobody reads), tokens past T to the last token (their LDS
    // rows are cleared before use).  A lane address is a per-lane base plus a wavefront-uniform
    // offset, all in 64 bits; only the last tile of a ragged T computes its own rows.
    // element loads: lane = column 64 c + lane of the tile, one row of t per instruction;
    // 16-byte loads: one instruction covers 256 / BM rows of t
    constexpr int kRowsPerVec = 256 / BM;
    const int vrow = lane / (BM / 4), vcol = (lane % (BM / 4)) * 4;
    const int64_t strideA = g.mxt ? 1 : sg.ldy, strideB = g.ldx;  // from one t to the next
    const float* laneA[kVecA ? 1 : F];
    const float* laneB[kVecB ? 1 : F];
    if (kVecA) {
        laneA[0] = sg.dY + (row0 + vcol < sg.rows ? row0 + vcol : 0);
    } else {
#pragma unroll
        for (int c = 0; c < F; ++c) {
            const int64_t j = row0 + c * 64 + lane < sg.rows ? row0 + c * 64 + lane : 0;
            const int64_t col = sg.idx ? sg.idx[j] : j;
            laneA[c] = sg.dY + (g.mxt ? col * sg.ldy : col);
        }
    }
    if (kVecB) {
        laneB[0] = g.X + (n0 + vcol < g.n ? n0 + vcol : 0);
    } else {
#pragma unroll
        for (int c = 0; c < F; ++c) laneB[c] = g.X + (n0 + c * 64 + lane < g.n ? n0 + c * 64 + lane : 0);
    }
    const uint32_t ring_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)ring));
    const int64_t vrowA = vrow * strideA, vrowB = vrow * strideB;
    // one 16-byte or 4-byte load instruction: `addr` per lane, LDS row r of the operand at `lds`
    auto load_vec = [&](const float* addr, uint32_t lds, int r) {
        asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off"
                     :
                     : "v"(addr), "s"(lds + r * BM * 4)
                     : "memory", "m0");
    };
    auto load_operand = [&](bool vec, const float* const* lanes, int64_t stride, int64_t vrow_off,
                            int t0, uint32_t lds) {
        if (vec) {
#pragma unroll
            for (int p = 0; p < F; ++p) {
                const int r0 = (p * 4 + wave) * kRowsPerVec;
                load_vec(lanes[0] + vrow_off + (t0 + r0) * stride, lds, r0);
            }
        } else {
#pragma unroll
            for (int p = 0; p < BK / 4; ++p) {
                const int r = p * 4 + wave;
                const int64_t uniform = (t0 + r) * stride;
#pragma unroll
                for (int c = 0; c < F; ++c) load4_to_lds(lanes[c] + uniform, lds + (r * BM + c * 64) * 4);
            }
        }
    };
    auto load_ragged = [&](bool vec, const float* const* lanes, int64_t stride, int t0, uint32_t lds) {
        if (vec) {
#pragma unroll
            for (int p = 0; p < F; ++p) {
                const int r0 = (p * 4 + wave) * kRowsPerVec;
                load_vec(lanes[0] + (r0 + vrow < T - t0 ? t0 + r0 + vrow : T - 1) * stride, lds, r0);
            }
        } else {
#pragma unroll
            for (int p = 0; p < BK / 4; ++p) {
                const int r = p * 4 + wave;
                const int64_t uniform = (r < T - t0 ? t0 + r : T - 1) * stride;
#pragma unroll
                for (int c = 0; c < F; ++c) load4_to_lds(lanes[c] + uniform, lds + (r * BM + c * 64) * 4);
            }
        }
    };
    auto issue = [&](int i) {
        const uint32_t st = ring_base + (i % kF32Stages) * 2 * kOperand * 4;
        const int t0 = t_begin + i * BK;
        if (T - t0 >= BK) {
            load_operand(kVecA, laneA, strideA, vrowA, t0, st);
            load_operand(kVecB, laneB, strideB, vrowB, t0, st + kOperand * 4);
        } else {
            load_ragged(kVecA, laneA, strideA, t0, st);
            load_ragged(kVecB, laneB, strideB, t0, st + kOperand * 4);
        }
    };

    const int wr = wave & 1, wc = wave >> 1;
    const int half = lane >> 5, l32 = lane & 31;
    const int offA = half * BM + wr * (BM / 2) + l32, offB = half * BN + wc * (BN / 2) + l32;

    f32x16 acc[F][F];
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
        for (int b = 0; b < F; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    constexpr int kAhead = kF32Stages - 1;
    for (int i = 0; i < kAhead && i < ntiles; ++i) issue(i);
    for (int i = 0; i < ntiles; ++i) {
        // tile i has landed once only the kAhead - 1 younger tiles are in flight; the loads issued
        // below overwrite the stage of tile i-1, whose LDS reads every wavefront has completed
        // (lgkmcnt) before the barrier
        if (i + kAhead - 1 < ntiles) wait_vmcnt<(kAhead - 1) * kLoads>(); else wait_vmcnt<0>();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        float* As = ring + (i % kF32Stages) * 2 * kOperand;
        float* Bs = As + kOperand;
        const int t0 = t_begin + i * BK;
        if (T - t0 < BK) {  // the last tile of a ragged T (the same branch for the whole workgroup)
            const int used = T - t0;
            for (int e = used * BM + tid; e < kOperand; e += 256) As[e] = Bs[e] = 0.f;
            __syncthreads();
        }
        // all fragments of the tile first, then its matrix instructions with the addresses and loads of
        // tile i + 3 among them (101 TFLOP/s with the loads issued before the reads)
        float fa[BK / 2][F], fb[BK / 2][F];
#pragma unroll
        for (int k = 0; k < BK / 2; ++k) {
#pragma unroll
            for (int a = 0; a < F; ++a) fa[k][a] = As[2 * k * BM + offA + a * 32];
#pragma unroll
            for (int b = 0; b < F; ++b) fb[k][b] = Bs[2 * k * BN + offB + b * 32];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < BK / 2; ++k) {
#pragma unroll
            for (int a = 0; a < F; ++a)
#pragma unroll
                for (int b = 0; b < F; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[k][a], fb[k][b], acc[a][b], 0, 0, 0);
            if (k == 1) {  // addresses and loads in the shadow of the matrix instructions
                __builtin_amdgcn_sched_barrier(0);
                if (i + kAhead < ntiles) issue(i + kAhead);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // accumulator element v of lane l is C[8*(v/4) + 4*(l/32) + v%4][l%32] of its fragment
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t row = row0 + wr * (BM / 2) + a * 32 + 8 * (v / 4) + 4 * half + (v % 4);
            if (row >= sg.rows) continue;
            const float s = !g.P && sg.rho ? sg.rho[row] : 1.0f;
#pragma unroll
            for (int b = 0; b < F; ++b) {
                const int64_t col = n0 + wc * (BN / 2) + b * 32 + l32;
                if (g.P) {
                    g.P[(static_cast<int64_t>(split) * g.Mp + sg.off + row) * g.Np + col] = acc[a][b][v];
                } else if (col < g.n) {
                    if (g.c_bf16) store_from_f32(static_cast<uint16_t*>(sg.C) + row * sg.ldc + col, s * acc[a][b][v]);
                    else store_from_f32(static_cast<float*>(sg.C) + row * sg.ldc + col, s * acc[a][b][v]);
                }
            }
        }
}

}  // namespace
}  // namespace grass
