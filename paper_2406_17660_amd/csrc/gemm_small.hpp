// bf16 MFMA GEMM with 128 x 128 tiles, register-staged: operands that load-to-LDS cannot fetch (rows on 2-byte
// boundaries, fewer than 32 tokens or 8 columns, 32-bit offsets that do not reach).
// Included by cgrad.hip only (device code shares one translation unit with its launchers).
#pragma once
#include "common.hpp"
#include "gemm_common.hpp"

namespace grass {
namespace {

// ------------------------------------------------------------------------------ bf16 MFMA GEMM
// 16 bytes from any element of a matrix (rows may start on 2-byte boundaries).
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(2))) Chunk16 { u32x4_t v; };

// One aligned 16-byte chunk (8 bf16) of row `krow` starting at column `col` of a [K x ncols] matrix
// (ncols a multiple of 8), zero outside the matrix.
__device__ __forceinline__ uint4 load_chunk(const uint16_t* __restrict__ base, int64_t ld,
                                            int64_t krow, int64_t col, int64_t K, int64_t ncols) {
    if (krow >= K || col >= ncols) return make_uint4(0, 0, 0, 0);
    return *reinterpret_cast<const uint4*>(base + krow * ld + col);
}

// v without its first `drop` (0..8) bf16 values, zeros moved in behind them.
__device__ __forceinline__ uint4 drop_elems(u32x4_t v, int drop) {
    unsigned long long lo = v[0] | (static_cast<unsigned long long>(v[1]) << 32);
    unsigned long long hi = v[2] | (static_cast<unsigned long long>(v[3]) << 32);
    if (drop & 4) { lo = hi; hi = 0; }
    const int bits = (drop & 3) * 16;
    lo = (lo >> bits) | ((hi << 1) << (63 - bits));
    hi >>= bits;
    if (drop & 8) { lo = 0; hi = 0; }
    return make_uint4(static_cast<uint32_t>(lo), static_cast<uint32_t>(lo >> 32),
                      static_cast<uint32_t>(hi), static_cast<uint32_t>(hi >> 32));
}

template <int BM_, int BN_, int BK_, int WR_, int WC_>
struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WR = WR_, WC = WC_;
    static constexpr int kThreads = 64 * WR * WC;
    static constexpr int WM = BM / WR, WN = BN / WC;  // wave tile
    static constexpr int FM = WM / 32, FN = WN / 32;  // 32x32 MFMA fragments per wave
    static constexpr int PAD = 16;                    // elements; keeps rows 32 B apart mod 128 B
    static constexpr int LDA = BM + PAD, LDB = BN + PAD;
    static constexpr int A_CHUNKS = BK * BM / 8 / kThreads;  // 16-byte chunks per thread
    static constexpr int B_CHUNKS = BK * BN / 8 / kThreads;
    static constexpr size_t kLdsBytes = static_cast<size_t>(BK) * (LDA + LDB) * 2;
    static constexpr int kWgPerCu = 2;
    static_assert(BK % 16 == 0 && WM % 32 == 0 && WN % 32 == 0, "tile shape");
    static_assert((BK * BM / 8) % kThreads == 0 && (BK * BN / 8) % kThreads == 0, "chunking");
};

// Operand fragment for v_mfma_f32_32x32x16_bf16 from a t-major LDS tile: lane l needs the 8
// values tile[k16 + 8*(l/32) + 0..7][c0 + l%32].  ds_read_b64_tr_b16 hands lane L of each
// 16-lane group the four values found at column (L%16) of the four rows addressed by lanes
// 4e + L/4... concretely: lane i of the group supplies the address of row (i/4), columns
// 4*(i%4)..+3, and receives column i of rows 0..3.  Two such reads give the 8 values.
__device__ __forceinline__ bf16x8 read_frag(const uint16_t* tile, int ld, int k16, int c0) {
    const int l = threadIdx.x & 63;
    const int L = l & 15;
    const int row = k16 + 8 * (l >> 5) + (L >> 2);
    const int col = c0 + 16 * ((l >> 4) & 1) + 4 * (L & 3);
    const uint16_t* p = tile + row * ld + col;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * ld));
    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
}

struct GemmArgs {
    const uint16_t* A;  // [K x Mcols], leading dimension lda
    const uint16_t* B;  // [K x Ncols], leading dimension ldb
    float* P;           // partials [S][Mp][Np], or the output itself (one slice, Np its leading dimension)
    int64_t lda, ldb, K, Mcols, Ncols, Mp, Np;
    int64_t out_rows, out_cols;  // of P: whole tiles, or the output's (not looked at by the staged 128 tile)
    int tiles_m, tiles_n, splits, ktiles_per_split;
    // row form of the left operand (large-tile kernel only): A is [rows of length K], row j of
    // the product is A + a_rows[j] * lda (a_rows == nullptr: row j itself)
    const int32_t* a_rows;
};

// The item (K slice and tile) of a workgroup of the 256-wide kernels; negative: none.  Consecutive
// items share a K slice and neighbouring tiles, and XCD x (workgroup b lands on XCD b % 8) is handed
// a contiguous range of them.
__device__ __forceinline__ int64_t work_item(const GemmArgs& g) {
    const int64_t items = static_cast<int64_t>(g.tiles_m) * g.tiles_n * g.splits;
    const int64_t chunk = (items + kNumXcd - 1) / kNumXcd;
    const int64_t item = static_cast<int64_t>(blockIdx.x % kNumXcd) * chunk + blockIdx.x / kNumXcd;
    return item < items ? item : -1;
}
// K tiles [begin, end) of slice `split`; `rows`: rows of the last of them (the others are whole).
struct KRange { int64_t begin, end; int rows; };
template <int BK>
__device__ __forceinline__ KRange k_range(const GemmArgs& g, int split) {
    const int64_t all = (g.K + BK - 1) / BK;
    KRange q;
    q.begin = static_cast<int64_t>(split) * g.ktiles_per_split;
    q.end = q.begin + g.ktiles_per_split < all ? q.begin + g.ktiles_per_split : all;
    q.rows = q.end > q.begin && q.end * BK > g.K ? static_cast<int>(g.K - (q.end - 1) * BK) : BK;
    return q;
}

// Stores a wavefront's block of FA x FB 32 x 32 accumulators at (m, n) of slice `split`.
template <int FA, int FB>
__device__ __forceinline__ void store_block(const GemmArgs& g, const f32x16 (&acc)[FA][FB], int split, int64_t m, int64_t n, int lane) {
    const int h = lane >> 5;
    float* P = g.P + (static_cast<int64_t>(split) * g.Mp + m) * g.Np + n;
    if (m + FA * 32 <= g.out_rows && n + FB * 32 <= g.out_cols) {
#pragma unroll
        for (int a = 0; a < FA; ++a)
#pragma unroll
            for (int b = 0; b < FB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = a * 32 + 8 * (v / 4) + 4 * h + (v % 4);
                    P[static_cast<int64_t>(row) * g.Np + b * 32 + (lane & 31)] = acc[a][b][v];
                }
        return;
    }
    const int64_t rows = g.out_rows - m, cols = g.out_cols - n - (lane & 31);  // an output of its own: its edge
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = a * 32 + 8 * (v / 4) + 4 * h + (v % 4);
            if (row >= rows) continue;
            float* dst = P + static_cast<int64_t>(row) * g.Np + (lane & 31);
#pragma unroll
            for (int b = 0; b < FB; ++b)
                if (b * 32 < cols) dst[b * 32] = acc[a][b][v];
        }
}

// kDense only tags the instantiation (dense full gradient vs compressed gradient) so that a
// profiler lists the two uses separately; the code is identical.
// kAnyAlign: operands whose rows, widths or bases break the aligned 16-byte chunks (about 10 %
// slower than the aligned form, which costs less than a copy of a wide operand).
template <typename Cfg, bool kDense, bool kAnyAlign>
__global__ __launch_bounds__(Cfg::kThreads) void tn_gemm_bf16_kernel(GemmArgs g) {
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    uint16_t* As = lds;
    uint16_t* Bs = lds + Cfg::BK * Cfg::LDA;

    // Work numbering: consecutive items share a K slice and neighbouring tiles.  Workgroup
    // b lands on XCD b % 8, so XCD x is handed the contiguous item range [x*chunk, (x+1)*chunk).
    const int64_t items = static_cast<int64_t>(g.tiles_m) * g.tiles_n * g.splits;
    const int64_t chunk = (items + kNumXcd - 1) / kNumXcd;
    const int64_t item = static_cast<int64_t>(blockIdx.x % kNumXcd) * chunk + blockIdx.x / kNumXcd;
    if (item >= items) return;
    const int tiles = g.tiles_m * g.tiles_n;
    const int split = static_cast<int>(item / tiles);
    const int tile = static_cast<int>(item % tiles);
    int tm, tn;
    tile_coords(tile, g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = static_cast<int64_t>(tm) * Cfg::BM, n0 = static_cast<int64_t>(tn) * Cfg::BN;
    const int64_t kt_begin = static_cast<int64_t>(split) * g.ktiles_per_split;
    const int64_t ktiles_all = (g.K + Cfg::BK - 1) / Cfg::BK;
    int64_t kt_end = kt_begin + g.ktiles_per_split;
    if (kt_end > ktiles_all) kt_end = ktiles_all;

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int wr = wave % Cfg::WR, wc = wave / Cfg::WR;

    f32x16 acc[Cfg::FM][Cfg::FN];
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // Global -> registers.  kAnyAlign: a thread fetches 16 bytes of the same columns in every row it
    // serves, from any element on; a chunk across the right edge is read from the last 8 columns and
    // one past it from the first (never outside a row), tokens past K from the last token; what
    // does not belong to the tile is dropped or zeroed on the way to LDS, in edge tiles only.
    u32x4_t ra[Cfg::A_CHUNKS], rb[Cfg::B_CHUNKS];
    constexpr int ACPR = Cfg::BM / 8, BCPR = Cfg::BN / 8;  // chunks per tile row
    static_assert(Cfg::kThreads % ACPR == 0 && Cfg::kThreads % BCPR == 0, "one column per thread");
    struct Side {
        const uint16_t* p;  // this thread's chunk in row 0
        int drop;           // leading values of the chunk that belong to the one before (8: all)
    };
    auto side = [&](const uint16_t* base, int64_t col, int64_t ncols) {
        Side q;
        q.drop = col >= ncols ? 8 : (col + 8 > ncols ? static_cast<int>(col + 8 - ncols) : 0);
        q.p = base + (q.drop == 0 ? col : (q.drop == 8 || ncols < 8 ? 0 : ncols - 8));
        return q;
    };
    const Side qa = side(g.A, m0 + (tid % ACPR) * 8, g.Mcols), qb = side(g.B, n0 + (tid % BCPR) * 8, g.Ncols);
    const bool edge = m0 + Cfg::BM > g.Mcols || n0 + Cfg::BN > g.Ncols;
    auto fetch_side = [&](u32x4_t& v, const uint16_t* base, const Side& q, int64_t ld, int64_t ncols,
                          int64_t row, int64_t col) {
        if (!kAnyAlign) {
            const uint4 w = load_chunk(base, ld, row, col, g.K, ncols);
            v = u32x4_t{w.x, w.y, w.z, w.w};
            return;
        }
        const uint16_t* p = q.p + (row < g.K ? row : g.K - 1) * ld;
        if (ncols >= 8) {
            v = reinterpret_cast<const Chunk16*>(p)->v;
        } else {  // fewer than 8 columns in all: element by element, from column 0
            uint16_t e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) e[i] = i < ncols ? p[i] : static_cast<uint16_t>(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = e[2 * i] | (static_cast<uint32_t>(e[2 * i + 1]) << 16);
        }
    };
    auto fetch = [&](int64_t kt) {
        const int64_t k0 = kt * Cfg::BK;
#pragma unroll
        for (int c = 0; c < Cfg::A_CHUNKS; ++c)
            fetch_side(ra[c], g.A, qa, g.lda, g.Mcols, k0 + (tid + c * Cfg::kThreads) / ACPR,
                       m0 + ((tid + c * Cfg::kThreads) % ACPR) * 8);
#pragma unroll
        for (int c = 0; c < Cfg::B_CHUNKS; ++c)
            fetch_side(rb[c], g.B, qb, g.ldb, g.Ncols, k0 + (tid + c * Cfg::kThreads) / BCPR,
                       n0 + ((tid + c * Cfg::kThreads) % BCPR) * 8);
    };
    auto fixed = [&](const u32x4_t& v, const Side& q, int64_t ncols, bool live) {
        return drop_elems(v, !live ? 8 : (ncols < 8 && q.drop < 8 ? 0 : q.drop));
    };
    auto stash = [&](int64_t kt) {
        const int64_t k0 = kt * Cfg::BK;
        const bool as_is = !kAnyAlign || (!edge && k0 + Cfg::BK <= g.K);
#pragma unroll
        for (int c = 0; c < Cfg::A_CHUNKS; ++c) {
            const int id = tid + c * Cfg::kThreads;
            uint4 v = make_uint4(ra[c][0], ra[c][1], ra[c][2], ra[c][3]);
            if (!as_is) v = fixed(ra[c], qa, g.Mcols, k0 + id / ACPR < g.K);
            *reinterpret_cast<uint4*>(As + (id / ACPR) * Cfg::LDA + (id % ACPR) * 8) = v;
        }
#pragma unroll
        for (int c = 0; c < Cfg::B_CHUNKS; ++c) {
            const int id = tid + c * Cfg::kThreads;
            uint4 v = make_uint4(rb[c][0], rb[c][1], rb[c][2], rb[c][3]);
            if (!as_is) v = fixed(rb[c], qb, g.Ncols, k0 + id / BCPR < g.K);
            *reinterpret_cast<uint4*>(Bs + (id / BCPR) * Cfg::LDB + (id % BCPR) * 8) = v;
        }
    };

    if (kt_begin < kt_end) {
        fetch(kt_begin);
        stash(kt_begin);
        __syncthreads();
        for (int64_t kt = kt_begin; kt < kt_end; ++kt) {
            const bool more = kt + 1 < kt_end;
            if (more) fetch(kt + 1);  // global loads in flight while the MFMAs run
#pragma unroll
            for (int k16 = 0; k16 < Cfg::BK; k16 += 16) {
                bf16x8 af[Cfg::FM], bfr[Cfg::FN];
#pragma unroll
                for (int i = 0; i < Cfg::FM; ++i)
                    af[i] = read_frag(As, Cfg::LDA, k16, wr * Cfg::WM + i * 32);
#pragma unroll
                for (int j = 0; j < Cfg::FN; ++j)
                    bfr[j] = read_frag(Bs, Cfg::LDB, k16, wc * Cfg::WN + j * 32);
#pragma unroll
                for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
                    for (int j = 0; j < Cfg::FN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j],
                                                                            acc[i][j], 0, 0, 0);
            }
            __syncthreads();
            if (more) {
                stash(kt + 1);
                __syncthreads();
            }
        }
    }

    // Partial tile -> P[split].  Accumulator element v of lane l is C[8*(v/4) + 4*(l/32) +
    // v%4][l%32] of its 32x32 fragment.  The partial buffer is padded to whole tiles.
    const int l = tid & 63;
    float* P = g.P + (static_cast<int64_t>(split) * g.Mp + m0 + wr * Cfg::WM) * g.Np + n0 +
               wc * Cfg::WN;
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = i * 32 + 8 * (v / 4) + 4 * (l >> 5) + (v % 4);
                P[static_cast<int64_t>(row) * g.Np + j * 32 + (l & 31)] = acc[i][j][v];
            }
}


}  // namespace
}  // namespace grass
