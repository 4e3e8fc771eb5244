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
    // moved to the left; its first `shift` columns repeat the chunk before it and are skipped.
    float* P = g.P + (static_cast<int64_t>(split) * g.Mp + m0 + wr * 128) * g.Np + n0 + wc * 128;
    const int shiftN = static_cast<int>(-g.Ncols & 7), shiftM = static_cast<int>(-g.Mcols & 7);
    const int edgeN = static_cast<int>((g.Ncols & ~int64_t{7}) - n0 - wc * 128);  // crossing chunk,
    const int edgeM = static_cast<int>((g.Mcols & ~int64_t{7}) - m0 - wr * 128);  // in this block
    if ((shiftN == 0 || edgeN >= 128 || edgeN <= -8) && (shiftM == 0 || edgeM >= 128 || edgeM <= -8)) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = a * 32 + 8 * (v / 4) + 4 * h + (v % 4);
                    P[static_cast<int64_t>(row) * g.Np + b * 32 + (lane & 31)] = acc[a][b][v];
                }
        return;
    }
    int col[4];  // where fragment column b goes, -1: nowhere
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        col[b] = b * 32 + (lane & 31);
        const int e = col[b] - edgeN;
        if (shiftN != 0 && e >= 0) col[b] = e < shiftN || e >= 8 ? -1 : col[b] - shiftN;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            int row = a * 32 + 8 * (v / 4) + 4 * h + (v % 4);
            const int e = row - edgeM;
            bool ok = true;
            if (shiftM != 0 && e >= 0) { ok = e >= shiftM && e < 8; row -= shiftM; }
            float* dst = P + static_cast<int64_t>(row) * g.Np;
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (ok && col[b] >= 0) dst[col[b]] = acc[a][b][v];
        }
}

}  // namespace
}  // namespace grass
