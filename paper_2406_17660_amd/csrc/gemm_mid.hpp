// bf16 MFMA GEMM with 128 x 256 and 128 x 128 tiles, load-to-LDS ring, two or three workgroups per
// compute unit: products whose height does not fill 256-row tiles, and those of few tiles.  Included by cgrad.hip only.
#pragma once
#include "gemm_large.hpp"

namespace grass {
namespace {

// The compressed products of small and odd ranks (r = 128, 300, 400 ...) waste up to half of a
// 256 x 256 tile.  This is the load-to-LDS kernel (gemm_large.hpp: same LDS permutation, transposing
// reads, hand-placed waits and fragment double-buffering) on a tile of 128 rows x 256 columns: four
// wavefronts of 64 x 128 (128 accumulator registers), K tiles of 32 in a ring of three 24 KB
// stages, so that two workgroups share a compute unit and fill each other's barriers.  Per flop it
// reads half as much again from LDS and from L2 as the 256 x 256 tile.  With two workgroups on every
// compute unit it reaches 0.82 - 0.87 of that kernel's rate (4096 x 4096, r = 1024, T = 131072: 1.16
// against 1.39 PFLOP/s; 2048 x 2048, r = 512, T = 65536: 1.01 against 1.16); the register-staged
// 128 x 128 kernel it replaces where both apply has one K tile in flight and reaches 0.60 - 0.66
// PFLOP/s there.
// Measured (whole steps, same K slices): 2048 x 2048, r = 300, T = 8192: 37 us, 45 with 128 x 128
// tiles; 488 x 8200, r = 122, T = 12224: 65 against 72; 4096 x 4096, r = 1024, T = 2048: 50
// against 54 with 256 x 256 tiles (256 workgroups instead of 128).
// BN = 128 is the same kernel on 128 x 128 tiles (wavefronts of 64 x 64, stages of 16 KB, three workgroups per
// compute unit).  It reads twice as much of the dense operand from L2 per flop as 128 x 256, so a filled chip
// prefers that one; a product that leaves compute units idle is bound by the time one workgroup takes per K
// tile, 0.39 us here, 0.34 + 0.2 u and 0.54 + 0.16 u us on the larger tiles at u workgroups per unit, and by
// starting up (3 - 6, 9 and 13 us).  (More stages for a workgroup that has a unit to itself change nothing: 48.8 us
// for 4096 x 4096, r = 1024, T = 2047 with three and with six.)  The register-staged kernel takes 0.5 - 0.7 us: 2360 x 416, r = 295, T = 674: 21.0 us
// per step with it, 18.5 with this; 440 x 272, r = 110, T = 9282: 22.2 and 20.2.
constexpr int kMidBM = 128, kMidBK = 32, kMidStages = 3;
constexpr int kMidAElems = kMidBK * kMidBM;
constexpr int mid_lds_bytes(int bn) { return kMidStages * kMidBK * (kMidBM + bn) * 2; }

__device__ __forceinline__ bf16x8 read_frag_swz128(const uint16_t* p) {  // rows of 128 elements
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * 128));
    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
}

// kDense only tags the instantiation for profilers (see gemm_small.hpp).
template <bool kDense, int BN>
__global__ __launch_bounds__(256, BN == 256 ? 2 : 3) void tn_gemm_bf16_mid_kernel(GemmArgs g) {
    constexpr int kMidBN = BN, NB = BN / 64;  // NB: fragments of B per wavefront, and loads of B per K tile
    constexpr int kMidStageElems = kMidBK * (kMidBM + kMidBN);
    constexpr int kMidLoads = 2 + NB;  // load-to-LDS instructions per wavefront and K tile
    constexpr int kRowsB = 2048 / BN;  // rows of B that the four wavefronts fill with one load each
    extern __shared__ __attribute__((aligned(1024))) uint16_t mid_ring[];

    const int64_t item = work_item(g);
    if (item < 0) return;
    const int tiles = g.tiles_m * g.tiles_n;
    const int split = __builtin_amdgcn_readfirstlane(static_cast<int>(item / tiles));
    const int tile = __builtin_amdgcn_readfirstlane(static_cast<int>(item % tiles));
    int tm, tn;
    tile_coords(tile, g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * kMidBM, n0 = static_cast<int64_t>(tn) * kMidBN;
    const KRange kr = k_range<kMidBK>(g, split);
    const int64_t kt_begin = kr.begin;
    const int ntiles = kr.end > kr.begin ? static_cast<int>(kr.end - kr.begin) : 0, last_rows = kr.rows;
    const int whole = last_rows == kMidBK ? ntiles : ntiles - 1;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave & 1, wc = wave >> 1;

    // ---- global -> LDS.  A: one load fills four rows of 16 slots, wavefront w rows 4w + 16 p;
    // B: the same, or with 256 columns two rows of 32 slots, rows 2w + 8 p.  The lane that fills physical slot s of row k
    // fetches
    // logical slot s ^ 4 (k % 4).  Columns past the edge are redirected to column 0.
    const int rowA = wave * 4 + (lane >> 4), rowB = wave * (kRowsB / 4) + lane / (BN / 8);
    int64_t colA = m0 + ((lane & 15) ^ (4 * (rowA & 3))) * 8, colB = n0 + ((lane % (BN / 8)) ^ (4 * (rowB & 3))) * 8;
    if (colA >= g.Mcols) colA = 0;
    if (colB >= g.Ncols) colB = 0;
    const uint16_t* gA = g.A + kt_begin * kMidBK * g.lda;
    const uint16_t* gB = g.B + kt_begin * kMidBK * g.ldb;
    const int64_t tileA = kMidBK * g.lda, tileB = kMidBK * g.ldb;
    uint32_t laneA[2], laneB[NB];
#pragma unroll
    for (int p = 0; p < 2; ++p) laneA[p] = static_cast<uint32_t>(((p * 16 + rowA) * g.lda + colA) * 2);
#pragma unroll
    for (int p = 0; p < NB; ++p) laneB[p] = static_cast<uint32_t>(((p * kRowsB + rowB) * g.ldb + colB) * 2);
    const uint32_t ring_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)mid_ring));
    auto issue_part = [&](uint32_t stage, int part) {  // parts 0, 1: A, 2..: B
        if (part < 2) load16_to_lds(gA, laneA[part], stage + (part * 16 + wave * 4) * 256);
        else load16_to_lds(gB, laneB[part - 2], stage + kMidAElems * 2 + ((part - 2) * kRowsB + wave * (kRowsB / 4)) * BN * 2);
    };
    auto stage_of = [&](int i) { return ring_base + (i % kMidStages) * kMidStageElems * 2; };
    auto issue = [&](int i) {  // any tile, the ragged last one included
        const uint32_t st = stage_of(i);
        if (i < whole) {
#pragma unroll
            for (int part = 0; part < kMidLoads; ++part) issue_part(st, part);
        } else {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int row = p * 16 + rowA, src = row < last_rows ? row : last_rows - 1;
                load16_to_lds(gA, static_cast<uint32_t>((src * g.lda + colA) * 2), st + (p * 16 + wave * 4) * 256);
            }
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                const int row = p * kRowsB + rowB, src = row < last_rows ? row : last_rows - 1;
                load16_to_lds(gB, static_cast<uint32_t>((src * g.ldb + colB) * 2),
                              st + kMidAElems * 2 + (p * kRowsB + wave * (kRowsB / 4)) * BN * 2);
            }
        }
        gA += tileA;
        gB += tileB;
    };
    // clears the rows of the ragged last tile that lie past K (after it has landed; ends in a barrier)
    auto clear_rows = [&](int i) {
        if (last_rows < kMidBK && i == ntiles - 1) {
            uint16_t* st = mid_ring + (i % kMidStages) * kMidStageElems;
            const uint4 zero = make_uint4(0, 0, 0, 0);
            for (int c = last_rows * 16 + tid; c < kMidBK * 16; c += 256) *reinterpret_cast<uint4*>(st + c * 8) = zero;
            for (int c = last_rows * (BN / 8) + tid; c < kMidBK * (BN / 8); c += 256)
                *reinterpret_cast<uint4*>(st + kMidAElems + c * 8) = zero;
            __syncthreads();
        }
    };

    // ---- LDS -> MFMA operand addressing (element offsets inside an operand block)
    const int L = lane & 15, g2 = (lane >> 4) & 1, h = lane >> 5;
    const int rrow = 8 * h + (L >> 2);
    const int swz = 4 * (L >> 2);
    const int lchunk = 2 * g2 + ((L & 3) >> 1);
    const int half = (L & 1) * 4;
    int offA[2], offB[NB];
#pragma unroll
    for (int a = 0; a < 2; ++a) offA[a] = rrow * 128 + ((((wr * 64 + a * 32) >> 3) ^ swz) + lchunk) * 8 + half;
#pragma unroll
    for (int b = 0; b < NB; ++b) offB[b] = rrow * BN + ((((wc * (BN / 2) + b * 32) >> 3) ^ swz) + lchunk) * 8 + half;

    f32x16 acc[2][NB];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    struct Frags { bf16x8 a[2], b[NB]; };
    auto read_b = [&](const uint16_t* sb, int b) {
        if constexpr (BN == 256) return read_frag_swz(sb + offB[b]);
        else return read_frag_swz128(sb + offB[b]);
    };
    auto read_half = [&](Frags& f, int stage, int k16, int part) {
        const uint16_t* sa = mid_ring + stage * kMidStageElems + k16 * 128;
        const uint16_t* sb = mid_ring + stage * kMidStageElems + kMidAElems + k16 * BN;
        if (part == 0) {
            f.a[0] = read_frag_swz128(sa + offA[0]);
#pragma unroll
            for (int b = 0; b < NB / 2; ++b) f.b[b] = read_b(sb, b);
        } else {
#pragma unroll
            for (int b = NB / 2; b < NB; ++b) f.b[b] = read_b(sb, b);
            f.a[1] = read_frag_swz128(sa + offA[1]);
        }
    };
    auto mfma_row = [&](const Frags& f, int a) {
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) {
            const int b = (a & 1) ? NB - 1 - bb : bb;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[a], f.b[b], acc[a][b], 0, 0, 0);
        }
    };
    // the matrix instructions of `cur` in two groups, each overlapped with half of the LDS reads of the
    // next slice; half of the loads of the tile two ahead
    // (`next_stage`: the ring stage of `next`'s tile)
    auto slice = [&](const Frags& cur, Frags& next, int next_stage, int next_k16, uint32_t stage, int part0,
                     bool do_load) {
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            read_half(next, next_stage, next_k16, part);
            mfma_row(cur, part);
            // 2 NB / 2 + 2 LDS reads among NB matrix instructions
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // DS read
            }
#pragma unroll
            for (int k = 2; k < NB; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (do_load) {
                if constexpr (NB == 4) {
                    issue_part(stage, part0 + part * 2);
                    if (part == 0) issue_part(stage, part0 + 1);
                } else {
                    issue_part(stage, part0 + part);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Software pipeline as in the 256 x 256 kernel, loads two tiles ahead:
    //   iteration i:  wait(tile i landed) ; barrier
    //                 MFMA on G = slice (i-1,1)  ||  F <- slice (i,0)  ||  half of tile i+2's loads
    //                 MFMA on F                  ||  G <- slice (i,1)  ||  the other half
    //   The loads overwrite the stage of tile i-1, whose last LDS reads were waited for before the
    //   barrier.
    constexpr int kAhead = kMidStages - 1;
    Frags F, G;
    if (ntiles > 0) {
        for (int i = 0; i < kAhead && i < ntiles; ++i) issue(i);
        if (ntiles > kAhead - 1) wait_vmcnt<(kAhead - 1) * kMidLoads>(); else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        clear_rows(0);
        read_half(F, 0, 0, 0);
        read_half(F, 0, 0, 1);
        if (kAhead < ntiles) issue(kAhead);
        read_half(G, 0, 16, 0);
        read_half(G, 0, 16, 1);
        __builtin_amdgcn_sched_barrier(0);
        mfma_row(F, 0);
        mfma_row(F, 1);
        __builtin_amdgcn_sched_barrier(0);
        int i = 1;
        auto step = [&](int stage) {  // a tile in ring stage `stage` (a constant at every call)
            wait_vmcnt<(kAhead - 1) * kMidLoads>();
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): own LDS reads of tile i-1 done
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t st = ring_base + (stage + kAhead) % kMidStages * kMidStageElems * 2;
            slice(G, F, stage, 0, st, 0, true);
            slice(F, G, stage, 16, st, kMidLoads / 2, true);
            gA += tileA;
            gB += tileB;
        };
        // once around the ring per turn: the stages are constants and so are the LDS addresses' offsets
        for (; i + 2 + kAhead < whole; i += kMidStages) {
            step(1);
            step(2);
            step(0);
        }
        int stage = 1;  // i % kMidStages
        for (; i + kAhead < whole; ++i) {
            step(stage);
            stage = stage == kMidStages - 1 ? 0 : stage + 1;
        }
        // drain: at most the ragged last tile is left to issue; wait for everything in flight
        for (; i < ntiles; ++i) {
            wait_vmcnt<0>();
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            if (i + kAhead < ntiles) issue(i + kAhead);
            clear_rows(i);
            slice(G, F, i % kMidStages, 0, 0, 0, false);
            slice(F, G, i % kMidStages, 16, 0, 0, false);
        }
        mfma_row(G, 0);
        mfma_row(G, 1);
    }

    store_block<2, NB>(g, acc, split, m0 + wr * 64, n0 + wc * (BN / 2), lane);
}

}  // namespace
}  // namespace grass
