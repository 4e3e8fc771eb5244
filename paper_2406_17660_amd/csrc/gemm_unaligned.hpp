// bf16 MFMA GEMM with 256 x 256 tiles for operands in any position: rows that start on 2-byte
// boundaries (odd widths, sliced tensors) and a K of any length.  Included by cgrad.hip only.
#pragma once
#include "gemm_large.hpp"

namespace grass {
namespace {

// The tile, the LDS permutation, the fragment reads and the order of the matrix instructions are
// those of the load-to-LDS kernel (gemm_large.hpp).  The load-to-LDS instruction needs 16-byte
// aligned rows, so here a tile goes through registers: 16-byte global loads that may start at any
// element, held for two K tiles, then written to one of two LDS stages.  Per K tile and
// wavefront that is 8 loads and 8 LDS writes, spread one pair per four matrix instructions
// (32 of them, 32 clocks each), which issue in their shadow.  The loads are ordinary ones (the
// compiler counts them), two tiles ahead: tile i+1 is written while tile i is multiplied and the
// registers it leaves receive tile i+3.
//
// Without it an odd-width operand has to be copied into padded rows first (T x 5461: 1.43 GB of
// traffic, 243 us at T = 65536, beside a product of 340 us).
//
// Edges.  A chunk of 8 columns that crosses the right edge of its matrix is loaded from the last 8
// columns instead (never past the end of a row, so never past the end of the matrix); the
// accumulator columns (rows, for the left operand) it feeds are stored where their true columns
// are.  Chunks wholly past the edge repeat column 0 and feed outputs that nobody reads.  Tokens
// past K are loaded as the last token and written to LDS as zeros.
// Requirements (checked by the launcher): at least 8 columns in each operand, element-aligned
// bases, 32-bit byte offsets inside a K tile.
__device__ __forceinline__ u32x4_t load16_any(const uint16_t* base, uint32_t lane_bytes) {
    return reinterpret_cast<const Chunk16*>(reinterpret_cast<const char*>(base) + lane_bytes)->v;
}

// Both operands in any position.
// kDense only tags the instantiation for profilers (see gemm_small.hpp).
template <bool kDense>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void tn_gemm_bf16_unaligned_kernel(GemmArgs g) {
    __shared__ __attribute__((aligned(1024))) uint16_t ring[2 * kFastStageElems];

    const int64_t item = work_item(g);
    if (item < 0) return;
    const int tiles = g.tiles_m * g.tiles_n;
    const int split = __builtin_amdgcn_readfirstlane(static_cast<int>(item / tiles));
    const int tile = __builtin_amdgcn_readfirstlane(static_cast<int>(item % tiles));
    int tm, tn;
    tile_coords(tile, g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * kFastBM, n0 = static_cast<int64_t>(tn) * kFastBN;
    const KRange kr = k_range<kFastBK>(g, split);
    const int64_t kt_begin = kr.begin;
    const int ntiles = kr.end > kr.begin ? static_cast<int>(kr.end - kr.begin) : 0, last_rows = kr.rows;
    const int whole = last_rows == kFastBK ? ntiles : ntiles - 1;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave & 1, wc = wave >> 1;

    // ---- global -> registers -> LDS: this lane fills physical slot `slot` of rows lrow + 8 p
    const int lrow = wave * 2 + (lane >> 5);
    const int slot = lane & 31;
    const int lchunk_g = slot ^ (4 * (lrow & 3));
    int64_t colA = m0 + lchunk_g * 8, colB = n0 + lchunk_g * 8;
    colA = colA >= g.Mcols ? 0 : (colA + 8 > g.Mcols ? g.Mcols - 8 : colA);
    colB = colB >= g.Ncols ? 0 : (colB + 8 > g.Ncols ? g.Ncols - 8 : colB);
    const uint16_t* gA = g.A + kt_begin * kFastBK * g.lda;
    const uint16_t* gB = g.B + kt_begin * kFastBK * g.ldb;
    const int64_t tileA = kFastBK * g.lda, tileB = kFastBK * g.ldb;
    uint32_t lane8[8];  // parts 0..3: rows lrow + 8 part of A, 4..7: of B
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        lane8[p] = static_cast<uint32_t>(((p * 8 + lrow) * g.lda + colA) * 2);
        lane8[4 + p] = static_cast<uint32_t>(((p * 8 + lrow) * g.ldb + colB) * 2);
    }
    uint16_t* const lds_lane = ring + lrow * 256 + slot * 8;
    // part `part` of tile i, whole tile (gA / gB point at it)
    auto load_part = [&](u32x4_t& r, const uint16_t* a, const uint16_t* b, int part) {
        r = load16_any(part < 4 ? a : b, lane8[part]);
    };
    auto write_part = [&](const u32x4_t& r, int i, int part) {
        *reinterpret_cast<u32x4_t*>(lds_lane + (i & 1) * kFastStageElems + (part >> 2) * kFastOperandElems +
                                    (part & 3) * 8 * 256) = r;
    };
    // any tile, ragged or not
    auto load_any = [&](u32x4_t (&r)[8], int i) {
        if (i < whole) {
#pragma unroll
            for (int part = 0; part < 8; ++part) load_part(r[part], gA, gB, part);
        } else if (i < ntiles) {
#pragma unroll
            for (int part = 0; part < 8; ++part) {
                const int row = (part & 3) * 8 + lrow;
                const int src = row < last_rows ? row : last_rows - 1;
                const uint32_t off = part < 4 ? static_cast<uint32_t>((src * g.lda + colA) * 2)
                                              : static_cast<uint32_t>((src * g.ldb + colB) * 2);
                const u32x4_t v = load16_any(part < 4 ? gA : gB, off);
                const u32x4_t zero = {0u, 0u, 0u, 0u};
                r[part] = row < last_rows ? v : zero;
            }
        }
        gA += tileA;
        gB += tileB;
    };
    auto write_all = [&](const u32x4_t (&r)[8], int i) {
#pragma unroll
        for (int part = 0; part < 8; ++part) write_part(r[part], i, part);
    };

    // ---- LDS -> MFMA operand addressing, as in the load-to-LDS kernel
    const int L = lane & 15, g2 = (lane >> 4) & 1, h = lane >> 5;
    const int rrow = 8 * h + (L >> 2);
    const int swz = 4 * (L >> 2);
    const int lchunk = 2 * g2 + ((L & 3) >> 1);
    const int half = (L & 1) * 4;
    int offA[4], offB[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        offA[i] = rrow * 256 + ((((wr * 128 + i * 32) >> 3) ^ swz) + lchunk) * 8 + half;
        offB[i] = rrow * 256 + ((((wc * 128 + i * 32) >> 3) ^ swz) + lchunk) * 8 + half;
    }

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    struct Frags { bf16x8 a[4], b[4]; };
    auto read_quarter = [&](Frags& f, int i, int k16, int part) {
        const uint16_t* sa = ring + (i & 1) * kFastStageElems + k16 * 256;
        const uint16_t* sb = sa + kFastOperandElems;
        if (part == 0) { f.a[0] = read_frag_swz(sa + offA[0]); f.b[0] = read_frag_swz(sb + offB[0]); }
        else if (part == 1) { f.b[1] = read_frag_swz(sb + offB[1]); f.b[2] = read_frag_swz(sb + offB[2]); }
        else if (part == 2) { f.b[3] = read_frag_swz(sb + offB[3]); f.a[1] = read_frag_swz(sa + offA[1]); }
        else { f.a[2] = read_frag_swz(sa + offA[2]); f.a[3] = read_frag_swz(sa + offA[3]); }
    };
    auto read_frags = [&](Frags& f, int i, int k16) {
#pragma unroll
        for (int part = 0; part < 4; ++part) read_quarter(f, i, k16, part);
    };
    auto mfma_row = [&](const Frags& f, int a) {
#pragma unroll
        for (int bb = 0; bb < 4; ++bb) {
            const int b = (a & 1) ? 3 - bb : bb;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[a], f.b[b], acc[a][b], 0, 0, 0);
        }
    };
    auto mfma16 = [&](const Frags& f) {
#pragma unroll
        for (int a = 0; a < 4; ++a) mfma_row(f, a);
    };
    // 16 matrix instructions of `cur` in four groups, each overlapped with a quarter of the LDS
    // reads of the next slice and followed by one LDS write of tile i+1 and one load of tile i+3
    auto slice = [&](const Frags& cur, Frags& next, int i, int next_k16, u32x4_t (&r)[8], int part0,
                     bool do_write, bool do_load) {
#pragma unroll
        for (int part = 0; part < 4; ++part) {
            read_quarter(next, i, next_k16, part);
            mfma_row(cur, part);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
            }
            __builtin_amdgcn_sched_barrier(0);
            if (do_write) write_part(r[part0 + part], i + 1, part0 + part);
            if (do_load) load_part(r[part0 + part], gA, gB, part0 + part);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto fence = [&]() {  // own LDS accesses done, then everybody's
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // Tile i+1 waits in R[(i+1) & 1] when iteration i begins.  Two stages suffice: iteration i
    // writes the stage of tile i-1, whose last reads were waited for before its barrier.
    Frags F, G;
    u32x4_t R0[8], R1[8];
    if (ntiles > 0) {
        int i = 1;
        if (whole > 5) {
            // Straight-line start and steady state: every path into the loop has the same loads in
            // flight, so that the compiler's wait before a write leaves the 15 younger ones alone.
            auto load_whole = [&](u32x4_t (&r)[8]) {
#pragma unroll
                for (int part = 0; part < 8; ++part) load_part(r[part], gA, gB, part);
                gA += tileA;
                gB += tileB;
            };
            load_whole(R0);
            load_whole(R1);
            write_all(R0, 0);
            load_whole(R0);
            fence();
            read_frags(F, 0, 0);
            read_frags(G, 0, 16);
            write_all(R1, 1);
            load_whole(R1);
            mfma16(F);
            __builtin_amdgcn_sched_barrier(0);
            // two tiles per turn; their loads (tiles i+3, i+4) are whole tiles
            for (; i + 4 < whole; i += 2) {
                fence();
                slice(G, F, i, 0, R0, 0, true, true);
                slice(F, G, i, 16, R0, 4, true, true);
                gA += tileA;
                gB += tileB;
                fence();
                slice(G, F, i + 1, 0, R1, 0, true, true);
                slice(F, G, i + 1, 16, R1, 4, true, true);
                gA += tileA;
                gB += tileB;
            }
        } else {
            load_any(R0, 0);
            load_any(R1, 1);
            write_all(R0, 0);
            load_any(R0, 2);
            fence();
            read_frags(F, 0, 0);
            read_frags(G, 0, 16);
            if (1 < ntiles) write_all(R1, 1);
            load_any(R1, 3);
            mfma16(F);
        }
        // the last tiles: loads of any kind, then none
        for (; i < ntiles; i += 2) {
            fence();
            slice(G, F, i, 0, R0, 0, i + 1 < ntiles, false);
            slice(F, G, i, 16, R0, 4, i + 1 < ntiles, false);
            load_any(R0, i + 3);
            if (i + 1 < ntiles) {
                fence();
                slice(G, F, i + 1, 0, R1, 0, i + 2 < ntiles, false);
                slice(F, G, i + 1, 16, R1, 4, i + 2 < ntiles, false);
                load_any(R1, i + 4);
            }
        }
        mfma16(G);
    }

    // Stores.  Only the tiles that hold a crossing chunk look at it: shift says how far the chunk was
    // moved to the left; its first `shift` columns repeat the chunk before it and are skipped.  (store_unaligned
    // below does the same; called here it costs this kernel 5 %: 300 x 1111, T = 65536: 116 us as it is, 121 so.)
    float* P = g.P + (static_cast<int64_t>(split) * g.Mp + m0 + wr * 128) * g.Np + n0 + wc * 128;
    const int shiftN = static_cast<int>(-g.Ncols & 7), shiftM = static_cast<int>(-g.Mcols & 7);
    const int edgeN = static_cast<int>((g.Ncols & ~int64_t{7}) - n0 - wc * 128);  // crossing chunk,
    const int edgeM = static_cast<int>((g.Mcols & ~int64_t{7}) - m0 - wr * 128);  // in this block
    if ((shiftN == 0 || edgeN >= 128 || edgeN <= -8) && (shiftM == 0 || edgeM >= 128 || edgeM <= -8)) {
        store_block<4, 4>(g, acc, split, m0 + wr * 128, n0 + wc * 128, lane);
        return;
    }
    int col[4];  // where fragment column b goes, -1: nowhere
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        col[b] = b * 32 + (lane & 31);
        const int e = col[b] - edgeN;
        if (shiftN != 0 && e >= 0) col[b] = e < shiftN || e >= 8 ? -1 : col[b] - shiftN;
        if (n0 + wc * 128 + col[b] >= g.out_cols) col[b] = -1;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            int row = a * 32 + 8 * (v / 4) + 4 * h + (v % 4);
            const int e = row - edgeM;
            bool ok = true;
            if (shiftM != 0 && e >= 0) { ok = e >= shiftM && e < 8; row -= shiftM; }
            ok = ok && m0 + wr * 128 + row < g.out_rows;
            float* dst = P + static_cast<int64_t>(row) * g.Np;
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (ok && col[b] >= 0) dst[col[b]] = acc[a][b][v];
        }
}

// Stores a wavefront's 128 x 128 block at (m, n).  Only the tiles that hold a crossing chunk look at it: shift
// says how far the chunk was moved to the left; its first `shift` columns repeat the chunk before it and are
// skipped.
__device__ __forceinline__ void store_unaligned(const GemmArgs& g, const f32x16 (&acc)[4][4], int split, int64_t m,
                                                int64_t n, int lane) {
    const int h = lane >> 5;
    float* P = g.P + (static_cast<int64_t>(split) * g.Mp + m) * g.Np + n;
    const int shiftN = static_cast<int>(-g.Ncols & 7), shiftM = static_cast<int>(-g.Mcols & 7);
    const int edgeN = static_cast<int>((g.Ncols & ~int64_t{7}) - n);  // crossing chunk,
    const int edgeM = static_cast<int>((g.Mcols & ~int64_t{7}) - m);  // in this block
    if ((shiftN == 0 || edgeN >= 128 || edgeN <= -8) && (shiftM == 0 || edgeM >= 128 || edgeM <= -8)) {
        store_block<4, 4>(g, acc, split, m, n, lane);
        return;
    }
    int col[4];  // where fragment column b goes, -1: nowhere
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        col[b] = b * 32 + (lane & 31);
        const int e = col[b] - edgeN;
        if (shiftN != 0 && e >= 0) col[b] = e < shiftN || e >= 8 ? -1 : col[b] - shiftN;
        if (n + col[b] >= g.out_cols) col[b] = -1;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            int row = a * 32 + 8 * (v / 4) + 4 * h + (v % 4);
            const int e = row - edgeM;
            bool ok = true;
            if (shiftM != 0 && e >= 0) { ok = e >= shiftM && e < 8; row -= shiftM; }
            ok = ok && m + row < g.out_rows;
            float* dst = P + static_cast<int64_t>(row) * g.Np;
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (ok && col[b] >= 0) dst[col[b]] = acc[a][b][v];
        }
}

// Left operand in aligned 16-byte chunks (a packed panel, or a dY whose rows are): it goes to LDS directly, into
// a ring of four stages, and only X passes through registers, four sets of them.  That halves the LDS writes and
// the loads that return to registers, which is what the kernel above loses against the load-to-LDS one: 2048 x
// 5461, r = 512, T = 65536 takes 342 us with it, 324 with this, 306 at the aligned width of 5464 (with none of the
// LDS writes at all it would be 316).
// The memory instructions are spread, at most one behind every two matrix instructions: the wavefronts of a
// workgroup share one address unit.  In clumps (a write and a load of X behind each of the first four groups of
// four, the left operand's loads behind the others) the same kernel takes 349 us; one write, one load behind
// every second group 329.
//
// Order of the memory instructions of a wavefront, B(i) = the four loads of X's tile i into set i % 4, A(i) = the
// four load-to-LDS of the left operand's: A(0) A(1) A(2) B(0) .. B(4), then in turns B(5) and A(3), B(6) and A(4),
// ...; iteration i begins when A(i) has landed, i.e. when at most B(i+3) A(i+1) B(i+4) A(i+2), as far as they exist,
// are outstanding, and writes B(i+1) to LDS.  The compiler counts the loads of X only, so its wait before a write
// (for all but 15) reaches back two tiles of both operands: as far as the loads of A are ahead.
// Taken from 64 K tiles per slice and for more than one row tile.  Shorter slices spend their time in the start and
// the end of this longer pipeline (3816 x 1881, r = 954, T = 5056, 20 tiles: 67.3 us per step with the kernel above,
// 70 with this); a single, mostly padded row tile is bound by the memory's time for X (4738 x 561, r = 70 columns,
// T = 112447: 289 and 296).  6288 x 9370, r = 786, T = 66176: 1224 us above, 1172 here.
constexpr int kUnalignedXMin = 64;
// kLeft: the left operand in any position and X in aligned chunks (a full gradient of odd height): the same with the
// operands' ways exchanged, taken by the same rule with columns for rows.  5461 x 2048, T = 65536: whole refresh steps
// 1351 -> 1274 us (with both operands through registers the product took 1290).  Full gradients in one slice, with both through
// registers / with this: 5461 x 2048 of 32 K tiles 33.0 / 34.2 us, 64: 52.9 / 53.0, 96: 73.0 / 72.1, 128: 92.9 / 91.1,
// 256: 182 / 168; 1021 x 4096 of 64: 52.6 / 53.6, 96: 70.9 / 70.1, 256: 164 / 154.  (Outputs of a few tiles gain from 4 K tiles on, but
// run on smaller tiles.)  A single column tile in many slices: 5461 x 256 in 12 of 128 K tiles 228 / 231.
template <bool kDense, bool kLeft = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void tn_gemm_bf16_unaligned_x_kernel(GemmArgs g) {
    constexpr int kStagesA = 4, kAheadA = 3;
    __shared__ __attribute__((aligned(1024))) uint16_t ringA[kStagesA * kFastOperandElems];
    __shared__ __attribute__((aligned(1024))) uint16_t ringB[2 * kFastOperandElems];
    // A and B below: the operand that goes to LDS directly and the one that passes through registers
    const int64_t lda = kLeft ? g.ldb : g.lda, ldb = kLeft ? g.lda : g.ldb;
    const int64_t colsA = kLeft ? g.Ncols : g.Mcols, colsB = kLeft ? g.Mcols : g.Ncols;

    const int64_t item = work_item(g);
    if (item < 0) return;
    const int tiles = g.tiles_m * g.tiles_n;
    const int split = __builtin_amdgcn_readfirstlane(static_cast<int>(item / tiles));
    const int tile = __builtin_amdgcn_readfirstlane(static_cast<int>(item % tiles));
    int tm, tn;
    tile_coords(tile, g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * kFastBM, n0 = static_cast<int64_t>(tn) * kFastBN;
    const KRange kr = k_range<kFastBK>(g, split);
    const int64_t kt_begin = kr.begin;
    const int ntiles = kr.end > kr.begin ? static_cast<int>(kr.end - kr.begin) : 0, last_rows = kr.rows;
    const int whole = last_rows == kFastBK ? ntiles : ntiles - 1;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave & 1, wc = wave >> 1;

    // ---- addressing: this lane fills physical slot `slot` of rows lrow + 8 p of either operand
    const int lrow = wave * 2 + (lane >> 5);
    const int slot = lane & 31;
    const int lchunk_g = slot ^ (4 * (lrow & 3));
    int64_t colA = (kLeft ? n0 : m0) + lchunk_g * 8, colB = (kLeft ? m0 : n0) + lchunk_g * 8;
    colA = colA >= colsA ? 0 : colA;
    colB = colB >= colsB ? 0 : (colB + 8 > colsB ? colsB - 8 : colB);
    const uint16_t* gA = (kLeft ? g.B : g.A) + kt_begin * kFastBK * lda;
    const uint16_t* gB = (kLeft ? g.A : g.B) + kt_begin * kFastBK * ldb;
    const int64_t tileA = kFastBK * lda, tileB = kFastBK * ldb;
    uint32_t laneA[4], laneB[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        laneA[p] = static_cast<uint32_t>(((p * 8 + lrow) * lda + colA) * 2);
        laneB[p] = static_cast<uint32_t>(((p * 8 + lrow) * ldb + colB) * 2);
    }
    const uint32_t ring_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)ringA)) + wave * 2 * 256 * 2;
    uint16_t* const lds_lane = ringB + lrow * 256 + slot * 8;
    auto stage_a = [&](int i) { return ring_base + (i % kStagesA) * kFastOperandElems * 2; };
    auto issue_a = [&](int i) {  // any tile
        const bool full = i < whole;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int row = p * 8 + lrow, src = row < last_rows ? row : last_rows - 1;
            load16_to_lds(gA, full ? laneA[p] : static_cast<uint32_t>((src * lda + colA) * 2), stage_a(i) + p * 8 * 256 * 2);
        }
        gA += tileA;
    };
    auto load_b = [&](u32x4_t (&r)[4], int i) {  // any tile; rows past K are zeros
        if (i < whole) {
#pragma unroll
            for (int p = 0; p < 4; ++p) r[p] = load16_any(gB, laneB[p]);
        } else {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int row = p * 8 + lrow, src = row < last_rows ? row : last_rows - 1;
                const u32x4_t v = load16_any(gB, static_cast<uint32_t>((src * ldb + colB) * 2));
                const u32x4_t zero = {0u, 0u, 0u, 0u};
                r[p] = row < last_rows ? v : zero;
            }
        }
        gB += tileB;
    };
    auto write_b = [&](const u32x4_t& r, int i, int p) {
        *reinterpret_cast<u32x4_t*>(lds_lane + (i & 1) * kFastOperandElems + p * 8 * 256) = r;
    };
    // clears the direct operand's rows of the ragged last tile that lie past K (after it has landed)
    auto clear_rows = [&](int i) {
        if (last_rows < kFastBK && i == ntiles - 1) {
            uint16_t* st = ringA + (i % kStagesA) * kFastOperandElems;
            const uint4 zero = make_uint4(0, 0, 0, 0);
            for (int c = last_rows * 32 + tid; c < kFastBK * 32; c += 256) *reinterpret_cast<uint4*>(st + c * 8) = zero;
            __syncthreads();
        }
    };

    // ---- LDS -> MFMA operand addressing, as in the load-to-LDS kernel
    const int L = lane & 15, g2 = (lane >> 4) & 1, h = lane >> 5;
    const int rrow = 8 * h + (L >> 2);
    const int swz = 4 * (L >> 2);
    const int lchunk = 2 * g2 + ((L & 3) >> 1);
    const int half = (L & 1) * 4;
    int offA[4], offB[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        offA[i] = rrow * 256 + ((((wr * 128 + i * 32) >> 3) ^ swz) + lchunk) * 8 + half;
        offB[i] = rrow * 256 + ((((wc * 128 + i * 32) >> 3) ^ swz) + lchunk) * 8 + half;
    }

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    struct Frags { bf16x8 a[4], b[4]; };
    auto read_quarter = [&](Frags& f, int i, int k16, int part) {
        const uint16_t* direct = ringA + (i % kStagesA) * kFastOperandElems + k16 * 256;
        const uint16_t* staged = ringB + (i & 1) * kFastOperandElems + k16 * 256;
        const uint16_t *sa = kLeft ? staged : direct, *sb = kLeft ? direct : staged;  // left operand, X
        if (part == 0) { f.a[0] = read_frag_swz(sa + offA[0]); f.b[0] = read_frag_swz(sb + offB[0]); }
        else if (part == 1) { f.b[1] = read_frag_swz(sb + offB[1]); f.b[2] = read_frag_swz(sb + offB[2]); }
        else if (part == 2) { f.b[3] = read_frag_swz(sb + offB[3]); f.a[1] = read_frag_swz(sa + offA[1]); }
        else { f.a[2] = read_frag_swz(sa + offA[2]); f.a[3] = read_frag_swz(sa + offA[3]); }
    };
    auto read_frags = [&](Frags& f, int i, int k16) {
#pragma unroll
        for (int part = 0; part < 4; ++part) read_quarter(f, i, k16, part);
    };
    auto mfma_row = [&](const Frags& f, int a) {
#pragma unroll
        for (int bb = 0; bb < 4; ++bb) {
            const int b = (a & 1) ? 3 - bb : bb;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[a], f.b[b], acc[a][b], 0, 0, 0);
        }
    };
    auto mfma_half = [&](const Frags& f, int a, int hf) {
#pragma unroll
        for (int bb = 2 * hf; bb < 2 * hf + 2; ++bb) {
            const int b = (a & 1) ? 3 - bb : bb;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[a], f.b[b], acc[a][b], 0, 0, 0);
        }
    };
    auto mfma16 = [&](const Frags& f) {
#pragma unroll
        for (int a = 0; a < 4; ++a) mfma_row(f, a);
    };
    // 16 matrix instructions of `cur` in pairs, every other one overlapped with a quarter of the LDS reads of the
    // next slice and each followed by `after(pair)`
    auto slice = [&](const Frags& cur, Frags& next, int i, int next_k16, auto after) {
#pragma unroll
        for (int part = 0; part < 4; ++part) {
            read_quarter(next, i, next_k16, part);
            mfma_half(cur, part, 0);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // DS read
            }
            __builtin_amdgcn_sched_barrier(0);
            after(2 * part);
            __builtin_amdgcn_sched_barrier(0);
            mfma_half(cur, part, 1);
            __builtin_amdgcn_sched_barrier(0);
            after(2 * part + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto fence = [&]() {  // own LDS accesses done, then everybody's
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // one iteration of the steady state: all tiles it loads are whole
    auto iteration = [&](Frags& F, Frags& G, u32x4_t (&r)[4], int i) {
        wait_vmcnt<16>();
        fence();
        auto memory = [&](int p) {  // after pair p of sixteen
            const int q = p / 4;
            if (p % 4 == 0) write_b(r[q], i + 1, q);
            else if (p % 4 == 1) r[q] = load16_any(gB, laneB[q]);
            else if (p % 4 == 3) load16_to_lds(gA, laneA[q], stage_a(i + kAheadA) + q * 8 * 256 * 2);
        };
        slice(G, F, i, 0, [&](int p) { memory(p); });
        slice(F, G, i, 16, [&](int p) { memory(8 + p); });
        gB += tileB;
        gA += tileA;
    };
    // one of the last
    auto last_iteration = [&](Frags& F, Frags& G, u32x4_t (&r)[4], int i) {
        switch (ntiles - i) {
            case 1: wait_vmcnt<0>(); break;
            case 2: wait_vmcnt<4>(); break;
            case 3: wait_vmcnt<8>(); break;
            case 4: wait_vmcnt<12>(); break;
            default: wait_vmcnt<16>();
        }
        fence();
        clear_rows(i);
        const bool more = i + 1 < ntiles;
        slice(G, F, i, 0, [&](int p) { if (more && p % 2 == 0) write_b(r[p / 2], i + 1, p / 2); });
        if (i + 5 < ntiles) load_b(r, i + 5);
        __builtin_amdgcn_sched_barrier(0);
        if (i + kAheadA < ntiles) issue_a(i + kAheadA);
        slice(F, G, i, 16, [&](int) {});
    };

    Frags F, G;
    u32x4_t R0[4], R1[4], R2[4], R3[4];
    if (ntiles > 0) {
        int i = 1;
        if (whole > 9) {  // straight line, so that every path into the loop has the same loads in flight
            auto load_whole = [&](u32x4_t (&r)[4]) {
#pragma unroll
                for (int p = 0; p < 4; ++p) r[p] = load16_any(gB, laneB[p]);
                gB += tileB;
            };
            auto issue_whole = [&](int t) {
#pragma unroll
                for (int p = 0; p < 4; ++p) load16_to_lds(gA, laneA[p], stage_a(t) + p * 8 * 256 * 2);
                gA += tileA;
            };
            for (int t = 0; t < kAheadA; ++t) issue_whole(t);
            load_whole(R0);
            __builtin_amdgcn_sched_barrier(0);
            load_whole(R1);
            __builtin_amdgcn_sched_barrier(0);
            load_whole(R2);
            __builtin_amdgcn_sched_barrier(0);
            load_whole(R3);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < 4; ++p) write_b(R0[p], 0, p);
            load_whole(R0);
            wait_vmcnt<16>();
            fence();
            read_frags(F, 0, 0);
            read_frags(G, 0, 16);
#pragma unroll
            for (int p = 0; p < 4; ++p) write_b(R1[p], 1, p);
            load_whole(R1);
            issue_whole(kAheadA);
            mfma16(F);
            __builtin_amdgcn_sched_barrier(0);
            for (; i + 8 < whole; i += 4) {
                iteration(F, G, R2, i);
                iteration(F, G, R3, i + 1);
                iteration(F, G, R0, i + 2);
                iteration(F, G, R1, i + 3);
            }
        } else {
            for (int t = 0; t < kAheadA && t < ntiles; ++t) issue_a(t);
            load_b(R0, 0);
            if (1 < ntiles) load_b(R1, 1);
            if (2 < ntiles) load_b(R2, 2);
            if (3 < ntiles) load_b(R3, 3);
#pragma unroll
            for (int p = 0; p < 4; ++p) write_b(R0[p], 0, p);
            if (4 < ntiles) load_b(R0, 4);
            wait_vmcnt<0>();
            fence();
            clear_rows(0);
            read_frags(F, 0, 0);
            read_frags(G, 0, 16);
            if (1 < ntiles) {
#pragma unroll
                for (int p = 0; p < 4; ++p) write_b(R1[p], 1, p);
            }
            if (5 < ntiles) load_b(R1, 5);
            __builtin_amdgcn_sched_barrier(0);
            if (kAheadA < ntiles) issue_a(kAheadA);
            mfma16(F);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (; i < ntiles; i += 4) {
            last_iteration(F, G, R2, i);
            if (i + 1 < ntiles) last_iteration(F, G, R3, i + 1);
            if (i + 2 < ntiles) last_iteration(F, G, R0, i + 2);
            if (i + 3 < ntiles) last_iteration(F, G, R1, i + 3);
        }
        mfma16(G);
    }
    store_unaligned(g, acc, split, m0 + wr * 128, n0 + wc * 128, lane);
}

}  // namespace
}  // namespace grass
