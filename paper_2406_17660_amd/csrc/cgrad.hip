// grass_compressed_grad and grass_dense_grad: C[j, i] = scale_j * sum_t dY[t, col_j] * X[t, i].
//
// Both operands are stored with the contraction index t as the ROW index (dY is T x m, X is
// T x n), i.e. this is a "TN" GEMM C = A^T B with A = dY[:, cols] and B = X.
//
// bf16 path (the hot one):
//   1. pack:   the r selected columns of dY are gathered once into a dense T x r_pad bf16
//              panel (zero padded to the tile width).  A per-element gather inside the
//              GEMM main loop would pull m/r times more cache lines through each CU's L1
//              than the tile uses; doing it once in an HBM-bound pass keeps the GEMM's
//              inner loop on full 16-byte loads.  (The dense gradient needs no pack.)
//              Wide matrices stage whole rows of dY through LDS (streaming loads, gather
//              from LDS); narrow sets of a group share one launch.  With dY stored m x T
//              there is no pack: the GEMM's tile loads fetch the selected rows themselves.
//   2. GEMM:   v_mfma_f32_32x32x16_bf16 tiles.  Global tiles [BK x BM] / [BK x BN] are staged
//              through LDS in their memory order (t-major) with 16-byte loads; the MFMA
//              operand layout (8 consecutive t per lane) is produced by the gfx950
//              transposing LDS read ds_read_b64_tr_b16, so no transpose is ever
//              materialised.  Split-K over T fills the 256 CUs; work items are numbered
//              so that the workgroups an XCD receives share one K slice (L2 reuse).
//   3. reduce: sums the split-K partials in a fixed order (deterministic), applies rho and
//              converts to the output dtype; in a regular step this, Adam and the update of
//              the rows of W are one kernel that reads the partial tiles directly.
// fp32 path: the same three stages without the pack, on operands split into bf16 parts or, for small
// products, on the fp32 matrix instruction (gemm_f32_split.hpp, gemm_f32.hpp).
#include <atomic>

#include "common.hpp"

#include "gemm_common.hpp"
#include "pack_kernels.hpp"
#include "gemm_small.hpp"
#include "gemm_large.hpp"
#include "gemm_unaligned.hpp"
#include "gemm_mid.hpp"
#include "gemm_gather_narrow.hpp"
#include "gemm_f32.hpp"
#include "gemm_f32_split.hpp"
#include "gemm_f32_short.hpp"
#include "reduce_kernels.hpp"

namespace grass {
namespace {

// ------------------------------------------------------------------------------ host side
using Cfg128 = TileCfg<128, 128, 64, 2, 2>;
enum TileId { kTile128 = 0, kTile256 = 1, kTileMid = 2 };  // mid: 128 x 256
constexpr int rows_log2(TileId id) { return id == kTile256 ? 8 : 7; }
constexpr int cols_log2(TileId id) { return id == kTile128 ? 7 : 8; }
constexpr int tile_rows(TileId id) { return 1 << rows_log2(id); }
constexpr int tile_k(TileId id) { return id == kTile128 ? Cfg128::BK : kFastBK; }
static_assert(kFastBM == 256 && kFastBN == 256 && kMidBM == 128 && kMidBK == kFastBK, "tile shapes");

// How the token dimension is divided: `splits` slices of `tokens` tokens, the last one shorter (it may end in a ragged
// K tile, whose missing tokens the kernels clear in LDS).
struct KSplit {
    int splits;
    int64_t tokens;
};
struct Plan {
    int64_t Mp, Np, rp;  // padded rows / cols of the partial buffer; packed panel width
    int tiles_m, tiles_n;
    size_t pack_bytes, partial_bytes;
};

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// A slice of partial tiles up to this size is re-read from the caches by the reduction.
constexpr int64_t kCachedSliceBytes = int64_t{16} << 20;

// The square tile that a product's K slices are planned for: 256 x 256 unless it wastes much of
// itself on padding.  (The kernel that runs may use another tile, see choose_plan: a slice's sums are
// taken in the same order whatever the tile, so results depend on the slices alone.)
TileId planned_tile(int64_t rows, int64_t n) {
    if (const int forced = test_option(GRASS_TEST_GEMM_TILE)) return forced == 256 ? kTile256 : kTile128;
    if (rows < 1 || n < 1) return kTile128;
    const double padded = static_cast<double>((rows + 255) / 256 * 256) * ((n + 255) / 256 * 256);
    return padded <= 1.35 * static_cast<double>(rows) * static_cast<double>(n) ? kTile256 : kTile128;
}

// The K tiles that slices are counted in: the large tile's whole ones (a ragged one ends the last slice), the small tile's all.
int64_t slice_tiles(TileId planned, int64_t T) {
    return planned == kTile256 ? T / kFastBK : (T + Cfg128::BK - 1) / Cfg128::BK;
}
KSplit in_slices(int64_t ktiles, int64_t slices, int bk) {
    int64_t per = (ktiles + slices - 1) / slices;
    if (per < 1) per = 1;
    const int splits = static_cast<int>((ktiles + per - 1) / per);
    return KSplit{splits < 1 ? 1 : splits, per * bk};
}

int64_t slice_count(TileId planned, int64_t T, int64_t rows, int64_t n) {
    const int edge = tile_rows(planned);
    const int64_t tm = (rows + edge - 1) >> rows_log2(planned), tn = (n + edge - 1) >> rows_log2(planned);
    const int64_t tiles = tm * tn;
    const int64_t ktiles = slice_tiles(planned, T);
    // Split K so that the workgroups fill whole rounds of the machine (256 CUs x workgroups
    // per CU) without paying too much for the partial tiles every slice adds.  In units of
    // the GEMM's time at full occupancy, c slices cost about 1 / fill(c) + c * k / T.  For
    // outputs of more than 16 MB per slice (the 7B / 13B layers) k = 1400: a slice writes and
    // re-reads 8 bytes per output element at ~4 TB/s while the GEMM spends 2 T flops per output
    // element at ~1.4 PFLOP/s.  The short, wide products of the small models are bound by
    // memory, not by the matrix cores, so an unfilled round costs them less and a slice
    // relatively more; k is then fitted to sweeps of the slice count on their layer shapes
    // (T = 65536): 2400 for the large tile (1024 x 1024 at r = 256: 42 slices, 81 us per step,
    // against 64 slices, 92 us) and 800 for the small one (512 x 512 at r = 128: 94 slices).
    // Each slice keeps at least 8 K tiles.
    const int slots_log2 = planned == kTile256 ? 8 : 9;
    int64_t smax = ktiles / 8 > 0 ? (ktiles / 8 < 128 ? ktiles / 8 : 128) : 1;
    if (const int cap = test_option(GRASS_TEST_MAX_K_SLICES)) smax = cap > 0 && cap < smax ? cap : smax;
    const bool cached = tm * edge * tn * edge * 4 <= kCachedSliceBytes;
    const double k = cached ? (planned == kTile256 ? 2400.0 : 800.0) : 1400.0;
    const double per_slice = k / static_cast<double>(T > 0 ? T : 1);
    int64_t s = 1;
    double best = 1e300;
    for (int64_t c = 1; c <= smax && tiles > 0; ++c) {
        const int64_t wgs = tiles * c, filled = ((wgs - 1) >> slots_log2) + 1;
        const double cost = static_cast<double>(filled << slots_log2) / static_cast<double>(wgs) + per_slice * c;
        if (cost < best - 1e-12) { best = cost; s = c; }
    }
    return s;
}

KSplit split_k(TileId planned, int64_t T, int64_t rows, int64_t n) {
    const int bk = tile_k(planned);
    return in_slices((T + bk - 1) / bk, slice_count(planned, T, rows, n), bk);
}

Plan make_plan(TileId id, const KSplit& k, int64_t T, int64_t rows, int64_t n, bool pack) {
    Plan p;
    p.tiles_m = static_cast<int>((rows + tile_rows(id) - 1) >> rows_log2(id));
    p.tiles_n = static_cast<int>((n + (1 << cols_log2(id)) - 1) >> cols_log2(id));
    p.Mp = static_cast<int64_t>(p.tiles_m) << rows_log2(id);
    p.Np = static_cast<int64_t>(p.tiles_n) << cols_log2(id);
    p.rp = p.Mp;
    p.pack_bytes = pack ? round_up(static_cast<size_t>(T) * p.rp * 2, 256) : 0;
    p.partial_bytes = static_cast<size_t>(k.splits) * p.Mp * p.Np * 4;
    return p;
}

// The GEMM kernels read the left operand as T x rows: a gather or the m x T storage needs the
// packing pass.
bool needs_pack(grass_dy_layout layout, bool gathered) {
    return gathered || layout == GRASS_DY_MxT;
}

// An operand whose width is not a multiple of 8 has rows that start on 2-byte boundaries.  Either
// the any-alignment form of the GEMM reads it where it is, or it is first copied into aligned rows
// (the left operand through the packing pass) for the faster aligned form.
struct Copies { bool a, b; };
// Measured: the any-alignment forms take 10 - 20 % longer than the aligned ones (1.3 PFLOP/s with
// the large tile, 0.45 with the small one), a copy moves 4 bytes per value at 5.2 TB/s and costs a
// launch; in the large tile the register route takes about 7 us more to fill and drain (2746 x 1509,
// r = 686, T = 448: 38.6 us in place, 35.1 with the copy), in the small one 4 (9576 x 371, r = 1024,
// T = 1472: 40.0 and 38.6).  2048 x 5461, r = 512, T = 65536:
// 429 us per step in place, 617 with the copy (split-K sum and Adam as two kernels in both; fused,
// the step in place takes 407); full gradient of 2807 x 6144, T = 5248: 224 us in
// place, 209 with the copy.  dY stored m x T is read row-wise by the aligned large tile without
// any pack, which the copy keeps possible.
Copies choose_copies(TileId tile, int64_t T, int64_t rows, int64_t n, grass_dy_layout layout, bool gathered) {
    const bool b_odd = n % 8 != 0, a_odd = !needs_pack(layout, gathered) && rows % 8 != 0;
    if (T < 1 || !(a_odd || b_odd) || test_option(GRASS_TEST_UNALIGNED_X) == 1) return Copies{false, false};
    if (layout == GRASS_DY_MxT && tile == kTile256 && T % kFastBK == 0) return Copies{false, b_odd};
    const double t = static_cast<double>(T);
    const double in_place = tile == kTile256 ? 7e-6 + 0.15 * 2.0 * t * rows * n / 1.3e15
                                             : 4e-6 + 0.15 * 2.0 * t * rows * n / 0.45e15;
    const double copied = (a_odd ? 4.0 * t * rows / 5.2e12 + 3e-6 : 0.0) + (b_odd ? 4.0 * t * n / 5.2e12 + 3e-6 : 0.0);
    return copied < in_place ? Copies{a_odd, b_odd} : Copies{false, false};
}
// What the launcher knows about the operands' positions: whole aligned 16-byte chunks (the left operand's after
// packing), and whether the copy kernel, which reads pairs of values, can read X.
struct Positions { bool a_chunks, x_chunks, x_pairs; };
Copies copies_at(TileId tile, int64_t T, int64_t rows, int64_t n, grass_dy_layout layout, bool gathered, const Positions& at) {
    const Copies c = choose_copies(tile, T, rows, n, layout, gathered);
    return c.b && !at.x_pairs ? Copies{false, false} : c;
}
size_t aligned_x_bytes(int64_t T, int64_t n) {
    return round_up(static_cast<size_t>(T) * ((n + 7) / 8 * 8) * 2, 256);
}

// Estimated time of a product's kernel in us.  A workgroup takes a time to start and to store its tile and, per K
// tile of 32 tokens, one that depends on how many workgroups a compute unit has, u = workgroups / 256.  `chunks`:
// load-to-LDS kernels (aligned operands), otherwise operands in any position through registers (one line for all three of
// the large tile's, which differ by 1 - 8 %).  No form falls when workgroups are added: slices are chosen by the least
// of these, and would be pushed past a fall for nothing.
double product_us(TileId id, bool chunks, bool row_form, double wgs, double ktiles) {
    const double u = wgs / 256.0;
    if (id == kTile256 && chunks) return (row_form ? 12.0 : 13.0) + ktiles * (u <= 1 ? 0.538 + 0.161 * u : 0.86 * ceil(u));
    if (id == kTile256) return 7.26 + ktiles * (u <= 1 ? 0.715 + 0.161 * u : 0.799 * ceil(u));
    if (id == kTileMid) return 9.06 + ktiles * (u <= 1 ? 0.338 + 0.2 * u : u <= 2 ? 0.967 : 0.581 * u);
    if (chunks) {
        const double many = 0.375 * u;
        return 2.83 + 3.17 * (u <= 1 ? u : 1) + ktiles * (u <= 1 ? 0.391 : u <= 2 ? 0.667 : many > 1.03 ? many : 1.03);
    }
    return 1.45 + ktiles * (u <= 2 ? 1.02 + 0.0872 * u : 0.586 * 2 * ceil(u / 2));
}
// A bf16 product as the launcher sees it.
struct Shape {
    int64_t T, rows, n;
    grass_dy_layout layout;
    bool gathered;
    bool row_form, pairs;  // the 256 tile gathers the rows of an m x T dY itself, 64 tokens per load
    Positions at;
    bool full_f32;  // a full gradient in fp32, which the product of one slice stores itself (but the staged 128 tile)
};
struct Choice { TileId tile; KSplit k; };
bool chunks_at(TileId id, const Shape& q, Copies* copy) {
    *copy = q.at.a_chunks && q.at.x_chunks ? Copies{false, false} : copies_at(id, q.T, q.rows, q.n, q.layout, q.gathered, q.at);
    return (q.at.a_chunks || copy->a) && (q.at.x_chunks || copy->b);
}
// The parts of a step's time that the tile and the slices decide, in us: the product, its partial tiles (written, then
// read by the reduction), and the passes that the tile needs ahead of it: dY stored m x T is packed (transposed) for all
// but the large tile, which gathers its rows itself, and an odd-width operand may be copied into aligned rows
// (choose_copies).  A full gradient's reduction is a launch more (3 us); stored by the product it takes the large tile
// 4.5 us where the output ends inside of it, next to nothing otherwise.  (The pack's terms are fitted with the others: they hold
// what else tells the packed products from the large tile's.)
struct TileTime {
    TileId id;
    bool chunks, row_form;
    double tiles, outputs, passes;
    bool stores;             // the product of one slice stores the full gradient itself
    double stored, reduced;  // us for that, and for the pass that it saves
    double us(double slices, double tokens) const {
        const double out = stores && slices == 1 ? stored : 1.45e-6 * outputs * slices + reduced;
        return passes + product_us(id, chunks, row_form, tiles * slices, tokens * (1.0 / kFastBK)) + out;
    }
};
TileTime tile_time(TileId id, const Shape& q) {
    Copies copy;
    TileTime r;
    r.id = id;
    r.chunks = chunks_at(id, q, &copy);
    r.row_form = q.row_form && id == kTile256 && r.chunks;
    const Plan p = make_plan(id, KSplit{1, 0}, q.T, q.rows, q.n, false);
    const double T = static_cast<double>(q.T);
    r.tiles = static_cast<double>(p.tiles_m) * p.tiles_n;
    r.outputs = static_cast<double>(p.Mp) * static_cast<double>(p.Np);
    r.passes = 0;
    if (copy.a) r.passes += 4.0 * T * static_cast<double>(q.rows) / 5.2e6 + 3;
    if (copy.b) {  // (one workgroup per row and 2048 columns)
        const double moved = 4.0 * T * static_cast<double>(q.n) / 5.2e6, groups = 2.8e-4 * T * static_cast<double>((q.n + 2047) / 2048);
        r.passes += (moved > groups ? moved : groups) + 3;
    }
    if (q.layout == GRASS_DY_MxT && !r.row_form) {
        const double moved = 2.0 * T * static_cast<double>(p.Mp + q.rows);
        r.passes += q.gathered ? moved / 1.13e6 + 9.04 : moved / 8.62e6 + 9.52;
    }
    r.stores = q.full_f32 && (id != kTile128 || r.chunks);
    r.stored = id == kTile256 && (q.rows % 128 != 0 || q.n % 128 != 0) ? 4.55 : 0.0;
    r.reduced = q.full_f32 ? 2.96 : 0.0;
    return r;
}
// What a plan needs of the workspace: packed panel, partial tiles and the aligned copy of X.
size_t choice_bytes(const Choice& c, const Shape& q) {
    Copies copy;
    const bool chunks = chunks_at(c.tile, q, &copy), row_form = q.row_form && c.tile == kTile256 && chunks;
    const Plan p = make_plan(c.tile, c.k, q.T, q.rows, q.n, !row_form && (needs_pack(q.layout, q.gathered) || copy.a));
    return p.pack_bytes + round_up(p.partial_bytes, 256) + (copy.b ? aligned_x_bytes(q.T, q.n) : 0);
}
// The tile and the K slices of a product, by estimated time.
//
// `k` are the slices planned for the square tile `planned`; of the tiles that run on them the quickest is taken.  Up
// to kJointMaxT tokens every tile is also tried with shorter slices of its own, down to two K tiles each, and taken if
// that is at least 5 % quicker: slices planned by how they fill the machine (split_k) know nothing of what starting a
// workgroup costs, nor which tile runs, and keep at least eight K tiles of the square one.  Longer slices are left out: the
// longer a sum in fp32 accumulators, the less exact (7833 x 2072, r = 334, T = 7833: 5 slices against 10).  Products of more
// tokens keep the slices of split_k and with them the order of their sums, in which one to ten of four million bf16 weights are rounded the
// other way: that is why the line lies there, and not for want of gain (1456 x 1800, r = 364, T = 128866: 335 us with split_k's, 292
// with slices of its own; 1200 x 9524, r = 300, T = 14720: 175 and 148).
// The estimates' constants are fitted to the steps of 590 random layers of up to 20000 tokens (all three tiles, up to
// 16 numbers of slices; both layouts, odd widths, rows and columns), 150 longer ones (tiles only) and 4200 full gradients
// of up to 9000 tokens.  The plan taken is 1.1 % from the best that is not left out for steps and 1.2 % for full gradients,
// 3.7 % before the estimate knew that one slice saves a pass (256 x 256, T = 256: 7.4 -> 4.9 us; 2064 x 608, m x T, T = 192:
// 14.6 -> 11.3; 3128 x 2736, T = 467: 22.9 -> 18.6; 1 % of them are slower by a tenth or more).  Whole steps
// against the tile alone: 352 x 8667, r = 88, T = 563: 29.7 -> 22.0 us; 302 x 1745, r = 37, T = 7341: 31.3 -> 25.3; 688 x 327,
// r = 172, T = 1924: 23.6 -> 19.3; 5848 x 744, r = 1024, T = 1523: 28.0 -> 25.0.  Longer slices left out cost full gradients most:
// 3608 x 1064, T = 960: 18 us in one slice, 30 in two.  Tiles of the longer layers: 0.3 % from the best.
constexpr int64_t kJointMaxT = 8192;
Choice choose_plan(TileId planned, const KSplit& k, const Shape& q, size_t room) {
    if (const int forced = test_option(GRASS_TEST_GEMM_TILE))
        return Choice{forced == 192 && q.at.a_chunks && q.at.x_chunks ? kTileMid : planned, k};
    const int run = test_option(GRASS_TEST_RUN_TILE);
    const bool aligned = q.at.a_chunks && q.at.x_chunks;
    Choice best{planned, k};
    TileTime times[3];
    int found = 0;
    double least = 1e300;
    for (const TileId id : {kTile256, kTileMid, kTile128}) {
        if (id == kTileMid && !aligned) continue;
        const TileTime& time = times[found++] = tile_time(id, q);
        if (id == kTile128 && planned == kTile256 && !time.chunks) continue;  // its K tiles are twice as long
        if (run == (id == kTile256 ? 256 : id == kTileMid ? 192 : 128)) return Choice{id, k};
        const double t = time.us(k.splits, static_cast<double>(k.tokens));
        if (t < least) { least = t; best.tile = id; }
    }
    if (run || q.T > kJointMaxT || test_option(GRASS_TEST_MAX_K_SLICES)) return best;
    least *= 0.95;
    for (int i = 0; i < found; ++i) {
        const TileTime& time = times[i];
        const uint32_t unit = (time.id == kTile128 && !time.chunks) || (time.row_form && q.pairs) ? 64 : 32;
        const uint32_t units = (static_cast<uint32_t>(q.T) + unit - 1) / unit, most = (static_cast<uint32_t>(q.T) + kFastBK - 1) / kFastBK / 2;
        uint32_t before = 0;
        for (const uint32_t c : {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 20, 24, 32, 42, 64}) {
            if (c > 1 && c > most) break;
            const uint32_t per = (units + c - 1) / c, slices = (units + per - 1) / per;
            if (slices == before) continue;
            before = slices;
            const int64_t tokens = static_cast<int64_t>(per) * unit;
            if ((tokens < q.T ? tokens : q.T) > k.tokens) continue;
            const double t = time.us(slices, static_cast<double>(tokens));
            if (!(t < least)) continue;
            const Choice other{time.id, KSplit{static_cast<int>(slices), tokens}};
            if (choice_bytes(other, q) <= room) { least = t; best = other; }
        }
    }
    return best;
}

// The addresses that a matrix of `rows` rows (at least one) takes up.
struct Span { uintptr_t begin, end; };
Span span_of(const void* p, int64_t rows, int64_t cols, int64_t ld, size_t elem) {
    const uintptr_t begin = reinterpret_cast<uintptr_t>(p);
    return Span{begin, begin + (static_cast<size_t>(rows - 1) * ld + cols) * elem};
}
bool overlap(const Span& a, const Span& b) { return a.begin < b.end && b.begin < a.end; }

// ---- narrow layers: the gather inside the GEMM (gemm_gather_narrow.hpp)
// Shapes the kernel takes, apart from what is asked of every set and of the addresses: at most two
// column tiles (beyond that each tile re-reads and re-gathers the rows of dY once more and the
// packed route wins: the step of a 512 x 1376 layer at r = 128, T = 65536 takes 83 us this way
// against 74), whole K tiles.
bool narrow_shape_ok(int64_t T, int64_t n, grass_dtype dt, grass_dy_layout layout) {
    return test_option(GRASS_TEST_NO_NARROW_GATHER) == 0 && test_option(GRASS_TEST_GEMM_TILE) == 0 &&
           dt == GRASS_BF16 && layout == GRASS_DY_TxM && T >= kNarrowBK && T % kNarrowBK == 0 &&
           n >= 8 && n % 8 == 0 && n <= 2 * kNarrowBN;
}
// one set: a single row tile, rows of dY that fit a stage
bool narrow_set_ok(int64_t rows, int64_t m_src) {
    return rows > 0 && rows <= kNarrowBM && m_src >= 8 && m_src % 8 == 0 && m_src <= kNarrowMaxM;
}
struct NarrowPlan {
    int64_t Mp, Np;
    int tiles_n, splits, ktiles_per_split;
};
// `tiles_m` row tiles in all, `panel_rows` rows of partial tiles per slice, `in_cols` = the row
// lengths of all inputs together (sum of m over the sets, plus n).  Slices: about two workgroups
// per compute unit (what the kernel's LDS use allows), as long as the partial tiles stay under a
// quarter of the input bytes (measured at the 60M shapes, T = 65536: 512 x 512 at r = 128 takes
// 26 us with 128 slices, 30 - 33 with 96, 170 or 256; the q/k/v group 66 us with 85 slices, 82
// with 42), every slice keeps at least four K tiles, and cap_bytes hold them.
// Up to kNarrowFitT tokens: the slices of least estimated time that fit `room`.  A round of workgroups (two per compute
// unit) takes 1.4 us and, per K tile of 16 tokens, 0.42 us and 0.34 times the workgroups per unit; a slice of partial
// tiles 0.27 us per MB.  Fitted to the steps of 110 random layers (one and three sets, 14 numbers of slices each), of
// which it is 1.1 % from the best.  Where those are longer than by the rule above (in 1 of 2000 random calls), the rule's are
// taken: a longer sum is less exact.  A quarter of the inputs' bytes allows a short product so few slices that most of
// the chip is idle.  512 x 512, r = 128, T = 1280: 29.7 -> 13.6 us, three of them, T = 2176: 51 -> 21; 256 x 256,
// r = 64, T = 256: 16.9 -> 11.1; 448 x 320, r = 56, T = 15552: 21.4 -> 17.7.  Longer layers keep their order of sums; the
// gain does not end at the line (512 x 512, r = 128: 108 slices and 25.7 us at T = 32768, 63 and 31.7 at T = 32784).
constexpr int64_t kNarrowFitT = 32768;
NarrowPlan narrow_plan(int64_t T, int64_t n, int tiles_m, int64_t panel_rows, int64_t in_cols,
                       size_t cap_bytes, size_t room) {
    NarrowPlan p;
    p.tiles_n = static_cast<int>((n + kNarrowBN - 1) / kNarrowBN);
    p.Np = static_cast<int64_t>(p.tiles_n) * kNarrowBN;
    p.Mp = (panel_rows + 7) / 8 * 8;
    const int64_t ktiles = T / kNarrowBK, tiles = static_cast<int64_t>(tiles_m) * p.tiles_n;
    const int64_t slice_bytes = p.Mp * p.Np * 4;
    int64_t s = tiles > 0 ? (512 + tiles - 1) / tiles : 1;
    const int64_t by_traffic = T * in_cols * 2 / 4 / (slice_bytes > 0 ? slice_bytes : 1);
    const int64_t by_space = static_cast<int64_t>(cap_bytes) / (slice_bytes > 0 ? slice_bytes : 1);
    s = s < by_traffic ? s : by_traffic;
    s = s < by_space ? s : by_space;
    s = s < ktiles / 4 ? s : ktiles / 4;
    s = s < 128 ? s : 128;
    if (const int cap = test_option(GRASS_TEST_MAX_K_SLICES)) s = cap > 0 && cap < s ? cap : s;
    s = s < 1 ? 1 : s;
    p.ktiles_per_split = static_cast<int>((ktiles + s - 1) / s);
    p.splits = static_cast<int>((ktiles + p.ktiles_per_split - 1) / p.ktiles_per_split);
    if (T > kNarrowFitT) return p;
    // the quickest that fit, unless they are longer than the above (which every accepted workspace holds)
    const int limit = test_option(GRASS_TEST_MAX_K_SLICES), longest = p.ktiles_per_split;
    int64_t quick_slices = 1, quick_per = ktiles;
    const size_t one = static_cast<size_t>(slice_bytes > 0 ? slice_bytes : 1);
    const int64_t fit = room / one < 128 ? static_cast<int64_t>(room / one) : 128;
    double least = 1e300;
    for (const int c : {1, 2, 3, 4, 5, 6, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64, 72, 85, 96, 112, 128}) {
        if (c > 1 && (2 * c > ktiles || (limit > 0 && c > limit))) break;
        const int64_t per = (ktiles + c - 1) / c, slices = (ktiles + per - 1) / per, wgs = tiles * slices;
        if (slices > 1 && slices > fit) break;
        const double u = static_cast<double>(wgs < 512 ? wgs : 512) / 256.0;
        const double us = static_cast<double>((wgs + 511) / 512) * (1.4 + static_cast<double>(per) * (0.42 + 0.34 * u)) +
                          0.27e-6 * static_cast<double>(slices * slice_bytes);
        if (us < least) {
            least = us;
            quick_slices = slices;
            quick_per = per;
        }
    }
    if (quick_per <= longest) {
        p.splits = static_cast<int>(quick_slices);
        p.ktiles_per_split = static_cast<int>(quick_per);
    }
    return p;
}

// ---- fp32 inputs (gemm_f32_split.hpp, gemm_f32.hpp, gemm_f32_short.hpp)
enum class F32Kernel { kSplit, kMfma, kShort };
enum class F32Tail { kNone, kRows, kCols };  // the rest of a regular step in the same call
struct F32Shape {
    int64_t T, n;
    int count;
    const int64_t* rows;  // of each set
    const int64_t* src;   // values per token of each set's dY; nullptr: not known (some workspace queries)
    grass_dy_layout layout;
    F32Tail tail;
    bool far;  // rows of T x m or T x n storage further apart than the kernels with split operands reach
};
struct F32Plan {
    F32Kernel kernel;
    int bm;  // tile edge
    int64_t Mp, Np;
    int tiles_m, tiles_n, splits, ktiles_per_split;
};
constexpr int64_t kF32SplitMinT = 1024;
// Below this many tokens the fp32 instruction, whose products are exact: split operands leave up to 2^-24 of a
// product out, which shows until the roundings of a longer sum outweigh it.  Error against 64 bits at 256 x 256, norm
// (and largest, over the sum of magnitudes), fp32 instruction / 64 tile / short kernel: T = 1: 2.5e-8 / 3.5e-8 / 4.2e-8
// (0.6e-7 / 1.4e-7 / 1.9e-7), T = 4: 4.0e-8 / 3.2e-8 / 4.1e-8 (1.7e-7 / 1.3e-7 / 1.7e-7), T = 8: 5.4e-8 / 3.1e-8 / 4.0e-8
// (2.2e-7 / 1.0e-7 / 1.3e-7).  A step of 32 rows takes 13.5 us so, 11 with the short kernel.
constexpr int64_t kF32PartsMinT = 8;

// The K slices of a product with this kernel and tile, those of least estimated time.  Split operands: a
// workgroup (one per compute unit) takes its slice in turns of two K tiles, and a turn takes so long.
// Columns gathered one by one cost the 64 tile more than its arithmetic does.  Measured per step, 128 / 64
// tile at the best slice count of each: 1024 x 1024, r = 256, T = 8192: 42 / 56 us (39 / 45 with dY stored
// m x T); 2048 x 2048, r = 256, T = 1024: 26 / 29 (22 / 20); 2048 x 512, r = 512, T = 512: 19 / 16 (18 /
// 15); 768 x 2000, r = 48, T = 8192: 40 / 44 (35 / 27).  The fp32 instruction: 150 TFLOP/s over the filled
// share of the machine's rounds.  A slice of partial tiles costs 8 bytes per output element at 4 TB/s, and
// every slice keeps at least four K tiles.  A call without a fused tail of fewer than 1024 tokens is not
// split, so that it needs no workspace: its K loop is short.
constexpr double f32_turn_us(int bm, bool mxt) { return bm == 128 ? (mxt ? 1.2 : 1.4) : (mxt ? 1.1 : 1.6); }
F32Plan f32_slices(F32Kernel kernel, int bm, const F32Shape& q, size_t cap_bytes) {
    int64_t total = 0, tm = 0;
    for (int i = 0; i < q.count; ++i) {
        total += (q.rows[i] + 7) / 8 * 8;
        tm += (q.rows[i] + bm - 1) / bm;
    }
    const int64_t tn = (q.n + bm - 1) / bm, T = q.T;
    F32Plan p;
    p.kernel = kernel;
    p.bm = bm;
    p.tiles_m = static_cast<int>(tm);
    p.tiles_n = static_cast<int>(tn);
    p.Mp = total;
    p.Np = (tn * bm + kF32Tile - 1) / kF32Tile * kF32Tile;  // a slice of any plan holds one of the fp32 instruction's
    p.splits = p.ktiles_per_split = 1;
    const int64_t bk = kernel == F32Kernel::kSplit ? f32_bk(bm) : kF32BK, ktiles = (T + bk - 1) / bk, tiles = tm * tn;
    const int64_t slice_bytes = p.Mp * p.Np * 4;
    const int64_t room = slice_bytes > 0 ? static_cast<int64_t>(cap_bytes) / slice_bytes : 1;
    int64_t smax = ktiles / 4;
    if (smax > 128) smax = 128;
    if (smax < 1 || (q.tail == F32Tail::kNone && T < kF32SplitMinT) || kernel == F32Kernel::kShort) smax = 1;
    if (const int cap = test_option(GRASS_TEST_MAX_K_SLICES)) smax = cap > 0 && cap < smax ? cap : smax;
    const double slice_us = static_cast<double>(slice_bytes) * 2 / 4e6;
    const double tile_us = 2.0 * static_cast<double>(T) * bm * bm / 150e6;  // on the whole machine
    double best = 1e300;
    for (int64_t c = 1; c <= smax && tiles > 0; ++c) {
        // slices of whole K tiles: the room must hold those that remain (a workspace of the size that
        // the unlimited plan asks for then gives that plan again)
        const int64_t per = (ktiles + c - 1) / c > 0 ? (ktiles + c - 1) / c : 1, slices = (ktiles + per - 1) / per;
        if (c > 1 && c > room && slices > room) break;
        const double rounds = static_cast<double>((tiles * c + 255) / 256);
        double cost = slice_us * static_cast<double>(c);
        if (kernel == F32Kernel::kMfma) cost += tile_us * rounds * 256 / static_cast<double>(c);
        else cost += rounds * static_cast<double>((per + 1) / 2) * f32_turn_us(bm, q.layout == GRASS_DY_MxT) + (bm == 128 ? 3 : 0);
        if (cost < best * (1 - 1e-9)) {
            best = cost;
            p.ktiles_per_split = static_cast<int>(per);
            p.splits = slices > 0 ? static_cast<int>(slices) : 1;
        }
    }
    return p;
}

// Cache lines of 128 bytes that the gather of a set touches per token (T x m storage).
int64_t f32_lines(int64_t rows, int64_t src) { return rows < (src + 31) / 32 ? rows : (src + 31) / 32; }

// The kernel of short products: all sets single row tiles, one round of workgroups (each has a compute unit to
// itself) or, with a fused tail, a second one that the longer product pays for; up to 512 tokens, the longest that
// sixteen wavefronts take in two turns.  A workgroup fetches its selected columns of dY by itself, which bounds it on
// inputs that no cache holds: steps of 0.60 times the time of the fp32 instruction's two launches below 2000 lines,
// 0.7 - 1.08 around 5000, 1.2 - 1.8 beyond 6000 (600 layers of r <= 32, T <= 512; 418 x 3224 tokens, r = 13: 11.8
// against 10.0 us, 343 x 142, r = 11: 7.1 and 10.4).  Column steps have their tail in launches of its own and gain
// less: 0.90 below 2000 lines, 0.98 - 1.25 around 4000.  A call without a tail, which the other kernels do not split,
// always gains (0.33 - 0.7 beyond 128 tokens).  Three sets of 8 rows, n = 8712, T = 4 (819 workgroups): 16 us against 9.
bool f32_short_shape(const F32Shape& q) {
    int64_t most = 0, sets = 0;
    for (int i = 0; i < q.count; ++i) {
        most = q.rows[i] > most ? q.rows[i] : most;
        sets += q.rows[i] > 0;
    }
    const int64_t tiles = sets * ((q.n + kShortTile - 1) / kShortTile);
    return most <= kShortTile && q.T <= 512 && (tiles <= 256 || (q.tail == F32Tail::kRows && q.T >= 64 && tiles <= 512));
}
bool f32_short_lines(const F32Shape& q) {
    if (q.tail == F32Tail::kNone || q.layout == GRASS_DY_MxT) return true;
    int64_t lines = 0;
    for (int i = 0; i < q.count; ++i) {
        const int64_t l = f32_lines(q.rows[i], q.src[i]);
        lines = l > lines ? l : lines;
    }
    return q.T * lines <= (q.tail == F32Tail::kRows ? 5120 : 2048);
}

// Estimated time in us, apart from what is the same for the fp32 instruction and the two tiles with split operands: a
// start, a time per K tile of a workgroup's slice (`alone`, and `shared` times the workgroups per compute unit), per
// 128 MB of gathered lines, per 10^6 bytes of partial tiles and per round of workgroups.  Fitted to 900 random
// layers between 0.1 and 30 Gflop (T 16 - 16384, r 1 - 4000, one to three sets, steps, separate calls, full gradients;
// every input new to the caches), which it meets within 7 % (median, 4 % with dY stored m x T).
double f32_us(const F32Plan& p, const F32Shape& q) {
    struct Cost { double start, alone, shared, lines, slices, round; };
    constexpr Cost kCosts[2][3] = {{{11.0, 0.19, 0.20, 0.024, 0.0, 0.0},     // T x m: the fp32 instruction
                                    {8.2, 0.18, 0.34, 0.033, 0.12, 3.2},     // split operands, 64 tile
                                    {8.8, 0.54, 0.067, 0.030, 0.34, 3.2}},   // 128 tile
                                   {{11.0, 0.21, 0.17, 0.12, 0.0, 0.0},      // m x T
                                    {7.7, 0.30, 0.23, 0.038, 0.43, 2.0},
                                    {7.6, 0.63, 0.040, 0.038, 0.36, 2.8}}};
    const bool mxt = q.layout == GRASS_DY_MxT;
    const Cost& k = kCosts[mxt][p.kernel == F32Kernel::kMfma ? 0 : p.bm == 64 ? 1 : 2];
    double lines = 0;
    for (int i = 0; i < q.count; ++i)
        lines += mxt ? static_cast<double>(q.rows[i]) * static_cast<double>((q.T + 31) / 32)
                     : static_cast<double>(f32_lines(q.rows[i], q.src[i])) * static_cast<double>(q.T);
    const double wgs = static_cast<double>(p.tiles_m) * p.tiles_n * p.splits, rounds = ceil(wgs / 256);
    return k.start + p.ktiles_per_split * (k.alone * rounds + k.shared * wgs / 256) + k.lines * lines * p.tiles_n * 128e-6 +
           k.slices * static_cast<double>(p.Mp * p.Np * 4) * p.splits * 1e-6 + k.round * rounds;
}

// The plans that this shape may get (one, or, where the source widths are not known, all that they decide
// between); returns how many.
int f32_candidates(const F32Shape& q, size_t cap_bytes, F32Plan (&c)[4]) {
    const auto one = [&](F32Kernel kernel, int bm) {
        c[0] = f32_slices(kernel, bm, q, cap_bytes);
        return 1;
    };
    const int forced = test_option(GRASS_TEST_GEMM_TILE);
    if (q.far || forced == 16) return one(F32Kernel::kMfma, kF32Tile);
    if (forced == kShortTile) return one(F32Kernel::kShort, kShortTile);
    if (forced) return one(F32Kernel::kSplit, forced == 64 ? 64 : 128);
    if (q.T < kF32PartsMinT) return one(F32Kernel::kMfma, kF32Tile);
    int found = 0;
    if (f32_short_shape(q)) {
        if (q.src && f32_short_lines(q)) return one(F32Kernel::kShort, kShortTile);
        if (!q.src) c[found++] = f32_slices(F32Kernel::kShort, kShortTile, q, cap_bytes);
    }
    const int first = found;
    c[found++] = f32_slices(F32Kernel::kMfma, kF32Tile, q, cap_bytes);
    // below 0.3 Gflop starting up is what costs, and the fp32 instruction starts sooner (680 x 288, r = 42, T = 1856:
    // 12.8 against 16.7 us with split operands, 959 x 1928, r = 119, T = 448, 0.2 Gflop: 15.9 and 17.4)
    int64_t total = 0;
    for (int i = 0; i < q.count; ++i) total += q.rows[i];
    if (2.0 * static_cast<double>(q.T) * static_cast<double>(total) * static_cast<double>(q.n) < 0.3e9) return found;
    c[found++] = f32_slices(F32Kernel::kSplit, 64, q, cap_bytes);
    c[found++] = f32_slices(F32Kernel::kSplit, 128, q, cap_bytes);
    if (!q.src) return found;
    // a fifth of a microsecond in favour of the fp32 instruction (90 other layers: 0.36 % above the best of the three,
    // 0.58 and 0.74 with nothing and with half a microsecond).  With split operands for everything beyond 0.3 Gflop
    // 1706 x 3400 (full gradient, T = 70) took 30.0 us, 22.6 with the fp32 instruction, and two sets of 28 of 304
    // columns, T = 16234, 100.5 with the 64 tile that a cost without the gather preferred, 35.1 with the 128 tile.
    int best = first;
    double least = f32_us(c[first], q) - 0.2;
    for (int i = first + 1; i < found; ++i) {
        const double us = f32_us(c[i], q);
        if (us < least) { least = us; best = i; }
    }
    c[0] = c[best];
    return 1;
}
F32Plan f32_plan(const F32Shape& q, size_t cap_bytes) {
    F32Plan c[4];
    f32_candidates(q, cap_bytes, c);
    return c[0];
}
// Workspace for the partial tiles of a product that is planned without a limit: a single slice without a fused
// tail has none (and is what the plan gives for no workspace too).
size_t f32_partial_bytes(const F32Shape& q) {
    F32Plan c[4];
    size_t most = 0;
    for (int i = f32_candidates(q, ~size_t{0} >> 1, c); i-- > 0;) {
        if (c[i].splits == 1 && q.tail == F32Tail::kNone) continue;
        const size_t bytes = static_cast<size_t>(c[i].splits) * c[i].Mp * c[i].Np * 4 + 256;
        most = bytes > most ? bytes : most;
    }
    return most;
}

// More than 64 KB of dynamic LDS has to be asked for, per kernel and device; the attribute sticks for
// the life of the process, so it is set once: a flag per device and kernel, set with release order
// after the attribute call has returned; two first callers both make the call.  `which`: a number
// per kernel.
hipError_t raise_lds_limit(const void* kernel, int bytes, int which) {
    static std::atomic<bool> raised[6][64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    if (dev >= 0 && dev < 64 && raised[which][dev].load(std::memory_order_acquire)) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && dev >= 0 && dev < 64) raised[which][dev].store(true, std::memory_order_release);
    return e;
}

void launch_f32_mfma(const F32Args& a, bool vec_a, bool vec_b, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const int64_t items = static_cast<int64_t>(a.tiles_m) * a.tiles_n * a.splits;
    const dim3 grid(static_cast<unsigned>((items + kNumXcd - 1) / kNumXcd * kNumXcd)), block(256);
    if (vec_a && vec_b) launch_stamped(tn_gemm_f32_mfma_kernel<true, true>, grid, block, 0, s, e0, e1, a);
    else if (vec_a) launch_stamped(tn_gemm_f32_mfma_kernel<true, false>, grid, block, 0, s, e0, e1, a);
    else if (vec_b) launch_stamped(tn_gemm_f32_mfma_kernel<false, true>, grid, block, 0, s, e0, e1, a);
    else launch_stamped(tn_gemm_f32_mfma_kernel<false, false>, grid, block, 0, s, e0, e1, a);
}

template <int BM, bool kMxT>
hipError_t launch_f32_split(const F32Args& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(tn_gemm_f32_split_kernel<BM, kMxT>),
                                         kF32LdsBytes, 2 + (BM == 128 ? 2 : 0) + (kMxT ? 1 : 0));
    if (e != hipSuccess) return e;
    const int64_t items = static_cast<int64_t>(a.tiles_m) * a.tiles_n * a.splits;
    const dim3 grid(static_cast<unsigned>((items + kNumXcd - 1) / kNumXcd * kNumXcd)), block(kF32Threads);
    launch_stamped(tn_gemm_f32_split_kernel<BM, kMxT>, grid, block, kF32LdsBytes, s, e0, e1, a);
    return hipSuccess;
}

template <typename Cfg, bool kDense, bool kAnyAlign>
hipError_t launch_gemm_kernel(const GemmArgs& g, unsigned grid, hipStream_t s) {
    auto kernel = tn_gemm_bf16_kernel<Cfg, kDense, kAnyAlign>;
    if (Cfg::kLdsBytes > 64 * 1024) {
        // set once per instantiation and device, as in raise_lds_limit
        static std::atomic<bool> raised[64];
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
        if (dev < 0 || dev >= 64 || !raised[dev].load(std::memory_order_acquire)) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     static_cast<int>(Cfg::kLdsBytes));
            if (e != hipSuccess) return e;
            if (dev >= 0 && dev < 64) raised[dev].store(true, std::memory_order_release);
        }
    }
    kernel<<<grid, Cfg::kThreads, Cfg::kLdsBytes, s>>>(g);
    return hipSuccess;
}

bool fused_stats_shape_ok(int64_t T, int64_t m, int64_t n, grass_dtype dt, grass_dy_layout layout,
                          int64_t ldy, int64_t ldx) {
    // the squares need complete sums, so the fused form cannot split K: it only pays when the
    // output tiles alone fill most of the 256 compute units
    const int64_t tiles = ((m + kFastBM - 1) / kFastBM) * ((n + kFastBN - 1) / kFastBN);
    const bool force = test_option(GRASS_TEST_FUSED_STATS) == 1;  // whenever the shape allows
    return (tiles >= 192 || force) && dt == GRASS_BF16 && layout == GRASS_DY_TxM && T >= kFastBK &&
           T % kFastBK == 0 &&
           m >= 8 && n >= 8 && m % 8 == 0 && n % 8 == 0 && ldy % 8 == 0 && ldx % 8 == 0 &&
           (kFastBK + 1) * ldy * 2 < (int64_t{1} << 32) && (kFastBK + 1) * ldx * 2 < (int64_t{1} << 32);
}

size_t fused_stats_bytes(int64_t m, int64_t n) {
    const int64_t tiles_m = (m + kFastBM - 1) / kFastBM, tiles_n = (n + kFastBN - 1) / kFastBN;
    return static_cast<size_t>(2 * tiles_n) * tiles_m * kFastBM * 4 + 256;
}

}  // namespace

size_t grad_row_stats_workspace_bytes(int64_t T, int64_t m, int64_t n, grass_dtype dt,
                                      grass_dy_layout layout, int64_t ldy, int64_t ldx) {
    if (fused_stats_shape_ok(T, m, n, dt, layout, ldy, ldx)) return fused_stats_bytes(m, n);
    // otherwise G is formed in fp32 inside the workspace and reduced from there
    return static_cast<size_t>(m) * n * 4 + 256 + gemm_workspace_bytes(T, m, n, dt, layout, false);
}

size_t grad_row_stats_least_bytes(int64_t T, int64_t m, int64_t n, grass_dtype dt,
                                  grass_dy_layout layout, int64_t ldy, int64_t ldx) {
    if (dt != GRASS_F32 && fused_stats_shape_ok(T, m, n, dt, layout, ldy, ldx)) return fused_stats_bytes(m, n);
    return static_cast<size_t>(m) * n * 4 + 256 +
           (dt == GRASS_F32 ? 0 : gemm_workspace_bytes(T, m, n, dt, layout, false, 0, true));
}

grass_status launch_grad_row_stats(const void* dY, grass_dy_layout layout, int64_t ldy,
                                   const void* X, int64_t ldx, grass_dtype dt, int64_t T, int64_t m,
                                   int64_t n, float* sumsq, void* ws, size_t ws_bytes,
                                   hipStream_t s) {
    if (m == 0) return GRASS_OK;
    char* base = static_cast<char*>(ws);
    base += (256 - reinterpret_cast<uintptr_t>(base) % 256) % 256;
    const bool fused = fused_stats_shape_ok(T, m, n, dt, layout, ldy, ldx) && aligned_to(dY, 16) &&
                       aligned_to(X, 16);
    if (fused) {
        if (ws_bytes < fused_stats_bytes(m, n)) return GRASS_ERR_WORKSPACE;
        GemmArgs g;
        g.A = static_cast<const uint16_t*>(dY);
        g.B = static_cast<const uint16_t*>(X);
        g.P = reinterpret_cast<float*>(base);
        g.lda = ldy; g.ldb = ldx; g.K = T; g.Mcols = m; g.Ncols = n;
        g.tiles_m = static_cast<int>((m + kFastBM - 1) / kFastBM);
        g.tiles_n = static_cast<int>((n + kFastBN - 1) / kFastBN);
        g.Mp = static_cast<int64_t>(g.tiles_m) * kFastBM;
        g.Np = static_cast<int64_t>(g.tiles_n) * kFastBN;
        g.out_rows = g.Mp;
        g.out_cols = g.Np;
        g.splits = 1;
        g.ktiles_per_split = static_cast<int>(T / kFastBK);
        g.a_rows = nullptr;
        const int64_t items = static_cast<int64_t>(g.tiles_m) * g.tiles_n;
        const int64_t chunk = (items + kNumXcd - 1) / kNumXcd;
        if (chunk * kNumXcd > 0x7FFFFFFF) return GRASS_ERR_SHAPE;
        tn_gemm_bf16_direct_kernel<true, true><<<static_cast<unsigned>(chunk * kNumXcd), 256, 0, s>>>(g);
        rowpart_reduce_kernel<<<static_cast<unsigned>((m + 255) / 256), 256, 0, s>>>(
            g.P, 2 * g.tiles_n, g.Mp, m, sumsq);
        return launch_status();
    }
    // G, then the product's own workspace (which starts at the next multiple of 256 bytes)
    const size_t g_bytes = static_cast<size_t>(m) * n * 4;
    if (ws_bytes < g_bytes + 256 + (dt == GRASS_F32 ? 0 : gemm_workspace_bytes(T, m, n, dt, layout, false, 0, true)))
        return GRASS_ERR_WORKSPACE;
    if (m > 65535) return GRASS_ERR_SHAPE;
    float* G = reinterpret_cast<float*>(base);
    const size_t rest = ws_bytes - static_cast<size_t>(base - static_cast<char*>(ws)) - g_bytes;
    const grass_status st = launch_tn_gemm(dY, layout, ldy, X, ldx, dt, T, m, n, nullptr, nullptr, G,
                                           GRASS_F32, n, base + g_bytes, rest, s, m);
    if (st != GRASS_OK) return st;
    return launch_row_stats(G, GRASS_F32, m, n, n, sumsq, s);
}

// The row-gathering kernel takes K tiles in pairs: every workgroup gets whole pairs.
static KSplit paired(KSplit k, int64_t T) {
    if (k.tokens % (2 * kFastBK) != 0) {
        k.tokens += kFastBK;
        k.splits = static_cast<int>((T + k.tokens - 1) / k.tokens);
    }
    return k;
}

double product_estimate_us(int tile, bool direct, int64_t workgroups, int64_t ktiles) {
    return product_us(tile == 256 ? kTile256 : tile == 192 ? kTileMid : kTile128, direct, false, static_cast<double>(workgroups),
                      static_cast<double>(ktiles));
}

// Bytes the narrow kernel's partial tiles may take: what a packed product with either square tile
// and one spare slice would.  gemm_workspace_bytes asks for as much wherever this kernel can run.
size_t narrow_cap_bytes(int64_t T, int64_t rows, int64_t n) {
    size_t cap = 0;
    for (const TileId id : {kTile128, kTile256}) {
        const KSplit k = in_slices(slice_tiles(id, T), slice_count(id, T, rows, n), tile_k(id));
        const Plan p = make_plan(id, k, T, rows, n, true);
        const size_t bytes = p.pack_bytes + static_cast<size_t>(k.splits + 1) * p.Mp * p.Np * 4;
        cap = bytes > cap ? bytes : cap;
    }
    return cap;
}

size_t gemm_workspace_bytes(int64_t T, int64_t mrows, int64_t n, grass_dtype dt,
                            grass_dy_layout layout, bool gathered, int64_t src_rows, bool least) {
    if (dt == GRASS_F32)
        return f32_partial_bytes(F32Shape{T, n, 1, &mrows, gathered ? &src_rows : &mrows, layout, F32Tail::kNone, false});
    // The launcher may plan for the small tile where the large one cannot be used, and run either plan
    // with any tile: room for the larger number of slices and the widest padding.
    const KSplit k1 = split_k(kTile128, T, mrows, n), k2 = split_k(kTile256, T, mrows, n);
    const int64_t slices = k1.splits > k2.splits ? k1.splits : k2.splits;
    const int64_t Mp = (mrows + 255) / 256 * 256, Np = (n + 255) / 256 * 256;
    bool pack = needs_pack(layout, gathered), copy_x = false;
    if (n % 8 != 0 || (!pack && mrows % 8 != 0)) {
        for (const TileId id : {kTile128, kTile256, kTileMid}) {
            const Copies copy = choose_copies(id, T, mrows, n, layout, gathered);
            pack = pack || copy.a;
            copy_x = copy_x || copy.b;
        }
    }
    size_t tiled = (pack ? round_up(static_cast<size_t>(T) * Mp * 2, 256) : 0) +
                         static_cast<size_t>(slices) * Mp * Np * 4 + (copy_x ? aligned_x_bytes(T, n) : 0);
    // what the launcher may choose instead wherever each operand lies (it keeps to the above without the room): more
    // slices, for 3 in 4 of 8000 random shapes at most 1.25 times the bytes of long slices, at most 7 times (1 -> 7 MB; 66 MB more)
    if (!least && T >= kFastBK && T <= kJointMaxT && mrows >= 8 && n >= 8) {
        const bool packed = needs_pack(layout, gathered), rows_form = layout == GRASS_DY_MxT && T % kFastBK == 0;
        const bool a_matters = !packed && mrows % 8 == 0;
        for (int where = 0; where < 8; ++where) {
            const bool a_off = where & 1, x_off = where & 2, row_form = where & 4, pairs = row_form && T % (2 * kFastBK) == 0;
            if ((a_off && !a_matters) || (row_form && !rows_form)) continue;
            for (const bool full_f32 : {false, true}) {
                if (full_f32 && gathered) continue;
                const Shape q{T, mrows, n, layout, gathered, row_form, pairs,
                              Positions{packed || (a_matters && !a_off), !x_off && n % 8 == 0, !x_off}, full_f32};
                for (const TileId planned : {kTile128, kTile256}) {
                    const KSplit k = planned == kTile128 ? k1 : pairs ? paired(k2, T) : k2;
                    const size_t bytes = choice_bytes(choose_plan(planned, k, q, ~size_t{0}), q);
                    tiled = bytes > tiled ? bytes : tiled;
                }
            }
        }
    }
    // the narrow kernel's slices are bounded by a cap of their own
    const bool narrow = gathered && narrow_shape_ok(T, n, dt, layout) && mrows <= GRASS_MAX_GROUP * kNarrowBM;
    size_t cap = narrow ? narrow_cap_bytes(T, mrows, n) : 0;
    if (narrow && !least && T <= kNarrowFitT) {
        // (the number of sets, one row tile each, is not known here)
        for (int sets = static_cast<int>((mrows + kNarrowBM - 1) / kNarrowBM); sets <= GRASS_MAX_GROUP; ++sets) {
            const NarrowPlan p = narrow_plan(T, n, sets, mrows, 0, cap, ~size_t{0});
            const size_t bytes = static_cast<size_t>(p.splits) * p.Mp * p.Np * 4;
            cap = bytes > cap ? bytes : cap;
        }
    }
    return (cap > tiled ? cap : tiled) + 256;
}

void gemm_plan_summary(int64_t T, int64_t m, int64_t rows, int count, int64_t n, grass_dtype dt,
                       grass_dy_layout layout, int* tile, int* k_slices) {
    if (dt == GRASS_F32) {
        int64_t each[GRASS_MAX_GROUP], src[GRASS_MAX_GROUP];  // the sets taken to be of equal size
        for (int i = 0; i < count; ++i) {
            each[i] = rows / count;
            src[i] = m > each[i] ? m : each[i];
        }
        const F32Plan p = f32_plan(F32Shape{T, n, count, each, src, layout, F32Tail::kNone, false}, ~size_t{0} >> 1);
        *tile = p.bm == 128 ? 128 : 64;
        *k_slices = p.splits;
        return;
    }
    if (m > 0 && count >= 1 && narrow_shape_ok(T, n, dt, layout) &&
        narrow_set_ok((rows / count + 7) / 8 * 8, m)) {  // the sets taken to be of equal size
        const size_t cap = narrow_cap_bytes(T, rows, n);
        const NarrowPlan p = narrow_plan(T, n, count, rows, m * count + n, cap, ~size_t{0});
        *tile = 0;
        *k_slices = p.splits;
        return;
    }
    TileId id = T >= kFastBK && rows >= 8 && n >= 8 ? planned_tile(rows, n) : kTile128;
    KSplit k = split_k(id, T, rows, n);
    // gathered rows, aligned operands; the rows of one set only are gathered by the product itself
    const bool row_form = layout == GRASS_DY_MxT && count == 1 && T % kFastBK == 0 && test_option(GRASS_TEST_PACK_MXT) == 0;
    const bool pairs = row_form && T % (2 * kFastBK) == 0 && test_option(GRASS_TEST_NO_PAIRS) == 0;
    if (id == kTile256 && pairs) k = paired(k, T);
    if (T >= kFastBK && rows >= 8 && n >= 8) {
        const Choice c = choose_plan(id, k, Shape{T, rows, n, layout, true, row_form, pairs, Positions{true, n % 8 == 0, true}, false},
                                     ~size_t{0});
        if (c.k.splits != k.splits || c.k.tokens != k.tokens) id = c.tile;  // slices of that tile's own
        k = c.k;
    }
    *tile = tile_rows(id);
    *k_slices = k.splits;
}

size_t gemm_group_workspace_bytes(int64_t T, const int64_t* rows, int count, int64_t n,
                                  grass_dtype dt, grass_dy_layout layout, bool step, bool least) {
    if (dt == GRASS_F32)
        return f32_partial_bytes(F32Shape{T, n, count, rows, nullptr, layout, step ? F32Tail::kRows : F32Tail::kNone, false});
    int64_t total = 0;
    size_t need = 0;  // the sets may also be run one at a time
    for (int i = 0; i < count; ++i) {
        total += (rows[i] + 7) / 8 * 8;
        const size_t one = gemm_workspace_bytes(T, rows[i], n, dt, layout, true, 0, least);
        need = one > need ? one : need;
    }
    const size_t joint = gemm_workspace_bytes(T, total, n, dt, layout, true, 0, least);
    return joint > need ? joint : need;
}

// Adam and the row update from a G_C that has been written to seg.C: fp32 steps whose workspace holds
// not one slice of partial tiles.
grass_status run_tail_unfused(const GemmSegment& q, int64_t n, hipStream_t s) {
    if (!q.tail || q.rows == 0) return GRASS_OK;
    const StepTail& t = *q.tail;
    if (t.U) {  // column form: Adam into U, then the update of the columns of W
        const grass_status st = launch_adam_rows(static_cast<const float*>(q.C), q.ldc, t.M, t.V, t.sdt,
                                                 q.rows, n, t.lr, t.beta1, t.beta2, t.eps, t.t, t.U, s);
        if (st != GRASS_OK) return st;
        return launch_scatter_cols(t.W, t.wdt, t.w_rows, t.ldw, q.idx, q.rho, t.alpha, t.U, q.rows, s);
    }
    return launch_adam_scatter(static_cast<const float*>(q.C), q.ldc, t.M, t.V, t.sdt, q.rows, n,
                               t.lr, t.beta1, t.beta2, t.eps, t.t, t.W, t.wdt, t.ldw, q.idx, q.rho,
                               t.alpha, s, t.step_scalars);
}

// What follows the matrix product for every set: the split-K reduction into the set's output,
// or, for a regular step, the fused reduction + Adam + update straight from the partial tiles
// [slices][Mp][Np] (the sets lie one after the other along the rows, each starting at a
// multiple of 8).
grass_status finish_segments(const GemmSegment* seg, int count, const float* partial, int slices,
                             int64_t Mp, int64_t Np, int64_t n, grass_dtype odt, hipStream_t s,
                             hipEvent_t ev_tail_start, hipEvent_t ev_tail_stop) {
    int64_t off = 0;
    // sets whose reduction, Adam and row update run as one kernel: a launch for those whose rows
    // allow wide accesses ([1]) and a launch for the others ([0])
    TailSets tails[2];
    int ntails[2] = {0, 0};
    const StepTail* tail_common[2] = {nullptr, nullptr};
    for (int i = 0; i < count; ++i) {
        const GemmSegment& q = seg[i];
        if (q.rows > 0 && q.tail) {
            const bool wide =
                reduce_adam_scatter_wide(*q.tail, n, q.c_wanted ? static_cast<float*>(q.C) : nullptr, q.ldc);
            // straight from the partial tiles; launched after the loop, together
            const TailSet one{partial + off * Np, q.rows, q.tail->M, q.tail->V, q.tail->W,
                              q.tail->ldw, q.idx, q.rho,
                              q.c_wanted ? static_cast<float*>(q.C) : nullptr, q.ldc, q.tail->U};
            if (q.tail->U) {  // column form: its own launch, followed by the column update
                TailSets single;
                single.set[0] = one;
                grass_status st = launch_reduce_adam_scatter(single, 1, wide, slices, Mp, Np, n, *q.tail, s,
                                                             ev_tail_start, ev_tail_stop);
                if (st != GRASS_OK) return st;
                st = launch_scatter_cols(q.tail->W, q.tail->wdt, q.tail->w_rows, q.tail->ldw, q.idx,
                                         q.rho, q.tail->alpha, q.tail->U, q.rows, s);
                if (st != GRASS_OK) return st;
            } else {
                tails[wide].set[ntails[wide]++] = one;
                tail_common[wide] = q.tail;
            }
        } else if (q.rows > 0) {
            const int64_t span = reduce_many(slices, Np) ? 256 : 256 * kReduceCols;
            const dim3 rgrid(static_cast<unsigned>((n + span - 1) / span), static_cast<unsigned>(q.rows));
            const float* part = partial + off * Np;
            if (reduce_many(slices, Np)) {
                if (odt == GRASS_F32)
                    splitk_reduce_many_kernel<float><<<rgrid, 256, 0, s>>>(
                        part, slices, Mp, Np, q.rows, n, q.rho, static_cast<float*>(q.C), q.ldc);
                else
                    splitk_reduce_many_kernel<uint16_t><<<rgrid, 256, 0, s>>>(
                        part, slices, Mp, Np, q.rows, n, q.rho, static_cast<uint16_t*>(q.C), q.ldc);
            } else if (odt == GRASS_F32)
                splitk_reduce_kernel<float><<<rgrid, 256, 0, s>>>(
                    part, slices, Mp, Np, q.rows, n, q.rho, static_cast<float*>(q.C), q.ldc);
            else
                splitk_reduce_kernel<uint16_t><<<rgrid, 256, 0, s>>>(
                    part, slices, Mp, Np, q.rows, n, q.rho, static_cast<uint16_t*>(q.C), q.ldc);
        }
        off += (q.rows + 7) / 8 * 8;
    }
    for (int wide = 1; wide >= 0; --wide) {
        if (ntails[wide] == 0) continue;
        const bool first = wide == 1 || ntails[1] == 0, last = wide == 0 || ntails[0] == 0;
        const grass_status st = launch_reduce_adam_scatter(
            tails[wide], ntails[wide], wide != 0, slices, Mp, Np, n, *tail_common[wide], s,
            first ? ev_tail_start : nullptr, last ? ev_tail_stop : nullptr);
        if (st != GRASS_OK) return st;
    }
    return launch_status();
}

// C_i = scale_i * (A_i^T X) for `count` row sets that share X.  The sets are packed side by
// side into one panel (each starts at a multiple of 8 columns), one GEMM covers the panel,
// and the partial tiles are reduced into each set's own output.
grass_status launch_tn_gemm_segments(const GemmSegment* seg, int count, grass_dy_layout layout,
                                     const void* X, int64_t ldx, grass_dtype dt, int64_t T,
                                     int64_t n, grass_dtype odt, void* ws, size_t ws_bytes,
                                     hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop,
                                     hipEvent_t ev_tail_start, hipEvent_t ev_tail_stop) {
    int64_t total = 0;  // panel columns in use
    for (int i = 0; i < count; ++i) {
        if (seg[i].rows > 65535) return GRASS_ERR_SHAPE;
        total += count > 1 ? (seg[i].rows + 7) / 8 * 8 : seg[i].rows;
    }
    if (total == 0 || n == 0) return GRASS_OK;
    if (dt == GRASS_F32) {
        int64_t rows[GRASS_MAX_GROUP], src[GRASS_MAX_GROUP];
        bool tails = false, cols = false, far = ldx >= kF32MaxStride;
        for (int i = 0; i < count; ++i) {
            rows[i] = seg[i].rows;
            src[i] = seg[i].src_rows;
            tails = tails || seg[i].tail != nullptr;
            cols = cols || (seg[i].tail && seg[i].tail->U);
            far = far || (layout == GRASS_DY_TxM && seg[i].ldy >= kF32MaxStride);
        }
        char* base = static_cast<char*>(ws);
        const size_t skip = base ? (256 - reinterpret_cast<uintptr_t>(base) % 256) % 256 : 0;
        const size_t cap = base && ws_bytes > skip ? ws_bytes - skip : 0;
        const F32Tail tail = cols ? F32Tail::kCols : tails ? F32Tail::kRows : F32Tail::kNone;
        const F32Plan p = f32_plan(F32Shape{T, n, count, rows, src, layout, tail, far}, cap);
        // partial tiles whenever something reads them: several slices, or a fused tail (which takes
        // the sums from there); a workspace that cannot hold even one slice leaves the direct form
        const bool partial = (p.splits > 1 || tails) &&
                             static_cast<size_t>(p.splits) * p.Mp * p.Np * 4 <= cap;
        F32Args a;
        bool vec_a = layout == GRASS_DY_TxM;
        int64_t off = 0;
        int tile0 = 0;
        for (int i = 0; i < count; ++i) {
            const GemmSegment& q = seg[i];
            a.set[i] = F32Set{static_cast<const float*>(q.dY), q.ldy, q.idx, q.rho, q.C, q.ldc, q.rows, off, tile0};
            vec_a = vec_a && !q.idx && aligned_to(q.dY, 16) && q.ldy % 4 == 0 && q.rows % 4 == 0;
            off += (q.rows + 7) / 8 * 8;
            tile0 += static_cast<int>((q.rows + p.bm - 1) / p.bm);
        }
        a.count = count;
        a.X = static_cast<const float*>(X);
        a.ldx = ldx; a.n = n; a.T = T;
        a.P = partial ? reinterpret_cast<float*>(base + skip) : nullptr;
        a.Mp = p.Mp; a.Np = p.Np;
        a.mxt = layout == GRASS_DY_MxT;
        a.c_bf16 = odt == GRASS_BF16;
        a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n;
        a.splits = p.splits; a.ktiles_per_split = p.ktiles_per_split;
        note_kernel(p.kernel == F32Kernel::kShort ? GRASS_KERNEL_F32_SHORT : p.kernel == F32Kernel::kMfma ? GRASS_KERNEL_F32
                    : p.bm == 64 ? GRASS_KERNEL_F32_SPLIT_64 : GRASS_KERNEL_F32_SPLIT_128);
        if (p.kernel == F32Kernel::kShort) {
            F32StepArgs q{};
            // one row tile per set, and nobody asks for the product's and the tail's own times
            bool fused = tails && !ev_start && !ev_stop && !ev_tail_start && !ev_tail_stop;
            for (int i = 0; i < count && fused; ++i) fused = seg[i].tail && !seg[i].tail->U && seg[i].rows <= kShortTile;
            if (fused) {
                for (int i = 0; i < count; ++i) {
                    const StepTail& t = *seg[i].tail;
                    q.set[i] = F32StepSet{t.M, t.V, t.W, t.ldw, seg[i].c_wanted ? static_cast<float*>(seg[i].C) : nullptr, seg[i].ldc};
                }
                const StepTail& t = *seg[0].tail;
                q.adam = make_params(t.lr, t.beta1, t.beta2, t.eps, t.t, t.step_scalars);
                q.alpha = t.alpha;
                q.s_bf16 = t.sdt == GRASS_BF16;
                q.w_bf16 = t.wdt == GRASS_BF16;
            }
            const int64_t tiles = static_cast<int64_t>(p.tiles_m) * p.tiles_n;
            if (tiles > 0x7FFFFFFF) return GRASS_ERR_SHAPE;
            const dim3 grid(static_cast<unsigned>(tiles)), block(kShortWaves * 64);
            if (fused) {
                if (a.mxt) tn_gemm_f32_short_kernel<true, true><<<grid, block, 0, s>>>(a, q);
                else tn_gemm_f32_short_kernel<false, true><<<grid, block, 0, s>>>(a, q);
                return launch_status();
            }
            if (a.mxt) launch_stamped(tn_gemm_f32_short_kernel<true, false>, grid, block, 0, s, ev_start, ev_stop, a, q);
            else launch_stamped(tn_gemm_f32_short_kernel<false, false>, grid, block, 0, s, ev_start, ev_stop, a, q);
        }
        hipError_t le = hipSuccess;
        if (p.kernel == F32Kernel::kMfma)
            launch_f32_mfma(a, vec_a, aligned_to(X, 16) && ldx % 4 == 0 && n % 4 == 0, s, ev_start, ev_stop);
        else if (p.kernel == F32Kernel::kSplit)
            le = p.bm == 128 ? (a.mxt ? launch_f32_split<128, true>(a, s, ev_start, ev_stop)
                                      : launch_f32_split<128, false>(a, s, ev_start, ev_stop))
                             : (a.mxt ? launch_f32_split<64, true>(a, s, ev_start, ev_stop)
                                      : launch_f32_split<64, false>(a, s, ev_start, ev_stop));
        if (le != hipSuccess) return GRASS_ERR_DEVICE;
        if (partial)
            return finish_segments(seg, count, a.P, p.splits, p.Mp, p.Np, n, odt, s, ev_tail_start, ev_tail_stop);
        if (ev_tail_start) (void)hipEventRecord(ev_tail_start, s);
        for (int i = 0; i < count; ++i) {
            const grass_status st = run_tail_unfused(seg[i], n, s);
            if (st != GRASS_OK) return st;
        }
        if (ev_tail_stop) (void)hipEventRecord(ev_tail_stop, s);
        return launch_status();
    }

    const bool gathered = count > 1 || seg[0].idx != nullptr;
    bool pack = needs_pack(layout, gathered);
    if (count > 1) {
        // One panel pays off while a slice of partial tiles of the joint problem still fits
        // the caches (fewer, fuller launches).  Beyond that every set fills the machine on its
        // own and the joint partial tiles would only spill to HBM: run the sets one by one.
        const TileId square = planned_tile(total, n);
        const Plan joint = make_plan(square, split_k(square, T, total, n), T, total, n, pack);
        if (joint.Mp * joint.Np * 4 > kCachedSliceBytes) {
            for (int i = 0; i < count; ++i) {
                // (timing hooks: the first set's GEMM and the last set's tail)
                const bool first = i == 0, last = i + 1 == count;
                const grass_status st = launch_tn_gemm_segments(
                    seg + i, 1, layout, X, ldx, dt, T, n, odt, ws, ws_bytes, s, first ? ev_start : nullptr,
                    first ? ev_stop : nullptr, last ? ev_tail_start : nullptr,
                    last ? ev_tail_stop : nullptr);
                if (st != GRASS_OK) return st;
            }
            return GRASS_OK;
        }
    }
    // Narrow layers (every set a single row tile of short dY rows): the gather runs inside the
    // GEMM, no panel is written.
    bool narrow = gathered && narrow_shape_ok(T, n, dt, layout) && aligned_to(X, 16) && ldx % 8 == 0 &&
                  ldx >= n && (kNarrowBK + 1) * ldx * 2 < (int64_t{1} << 32);
    for (int i = 0; i < count && narrow; ++i)
        narrow = seg[i].idx && narrow_set_ok(seg[i].rows, seg[i].src_rows) && aligned_to(seg[i].dY, 16) &&
                 seg[i].ldy % 8 == 0 && seg[i].ldy >= seg[i].src_rows &&
                 (kNarrowBK + 1) * seg[i].ldy * 2 < (int64_t{1} << 32);
    if (narrow) {
        char* base = static_cast<char*>(ws);
        const size_t skip = (256 - reinterpret_cast<uintptr_t>(base) % 256) % 256;
        base += skip;
        const size_t room = ws_bytes > skip ? ws_bytes - skip : 0;
        NarrowArgs a;
        int64_t in_cols = n;
        int off = 0;
        for (int i = 0; i < count; ++i) {
            a.set[i] = NarrowSet{static_cast<const uint16_t*>(seg[i].dY), seg[i].ldy, seg[i].idx,
                                 static_cast<int>(seg[i].rows), static_cast<int>(seg[i].src_rows / 8), off, i};
            off += static_cast<int>((seg[i].rows + 7) / 8 * 8);
            in_cols += seg[i].src_rows;
        }
        const size_t cap = narrow_cap_bytes(T, total, n);
        const NarrowPlan np = narrow_plan(T, n, count, off, in_cols, cap, room);
        if (static_cast<size_t>(np.splits) * np.Mp * np.Np * 4 > room) return GRASS_ERR_WORKSPACE;
        a.count = count;
        a.X = static_cast<const uint16_t*>(X);
        a.ldx = ldx;
        a.n = n;
        a.P = reinterpret_cast<float*>(base);
        a.Mp = np.Mp;
        a.Np = np.Np;
        a.ktiles = T / kNarrowBK;
        a.tiles_m = count;
        a.tiles_n = np.tiles_n;
        a.splits = np.splits;
        a.ktiles_per_split = np.ktiles_per_split;
        const int64_t items = static_cast<int64_t>(count) * np.tiles_n * np.splits;
        const unsigned grid = static_cast<unsigned>((items + kNumXcd - 1) / kNumXcd * kNumXcd);
        {   // more than 64 KB of LDS: the attribute is set once per device (see raise_lds_limit)
            static std::atomic<bool> raised[64];
            int dev = 0;
            if (hipGetDevice(&dev) != hipSuccess) return GRASS_ERR_DEVICE;
            if (dev < 0 || dev >= 64 || !raised[dev].load(std::memory_order_acquire)) {
                if (hipFuncSetAttribute(reinterpret_cast<const void*>(tn_gemm_gather_narrow_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize,
                                        kNarrowLdsBytes) != hipSuccess)
                    return GRASS_ERR_DEVICE;
                if (dev >= 0 && dev < 64) raised[dev].store(true, std::memory_order_release);
            }
        }
        note_kernel(GRASS_KERNEL_NARROW);
        launch_stamped(tn_gemm_gather_narrow_kernel, dim3(grid), dim3(256), kNarrowLdsBytes, s, ev_start,
                       ev_stop, a);
        return finish_segments(seg, count, a.P, np.splits, np.Mp, np.Np, n, odt, s, ev_tail_start,
                               ev_tail_stop);
    }
    const void* dY0 = seg[0].dY;  // read directly by the GEMM only when nothing is packed
    const int64_t ldy0 = seg[0].ldy;
    // K slices: planned for the large tile where it can be used at all
    TileId planned = planned_tile(total, n);
    bool sizes;  // what the 256-wide kernels ask for: per-lane byte offsets inside a K tile in 32 bits
    {
        const int64_t panel_ld = (total + kFastBM - 1) / kFastBM * kFastBM;
        const int64_t lda_max = pack || panel_ld > ldy0 ? panel_ld : ldy0;
        sizes = (kFastBK + 1) * lda_max * 2 < (int64_t{1} << 32) &&
                (kFastBK + 1) * ldx * 2 < (int64_t{1} << 32) && T >= kFastBK && total >= 8 && n >= 8;
        const bool a_ok = pack || total % 8 != 0 || (aligned_to(dY0, 16) && ldy0 % 8 == 0);
        const bool b_ok = n % 8 != 0 ? aligned_to(X, 4) : aligned_to(X, 16) && ldx % 8 == 0;
        if (!(a_ok && b_ok && sizes)) planned = kTile128;
    }
    KSplit ks = split_k(planned, T, total, n);
    // dY stored m x T: the selected rows are contiguous, so the large-tile kernel can gather them
    // itself (no packing pass) when K is whole tiles and its 32-bit row offsets reach every row
    const int64_t src_rows = seg[0].idx ? seg[0].src_rows : total;
    const bool rows_ok = layout == GRASS_DY_MxT && count == 1 && sizes && T % kFastBK == 0 &&
                         aligned_to(dY0, 16) && ldy0 % 8 == 0 && src_rows > 0 &&
                         src_rows * ldy0 * 2 + 128 < (int64_t{1} << 32) && test_option(GRASS_TEST_PACK_MXT) == 0;
    // whole cache lines per row (64 values of k per load) when the K tiles pair up
    const bool pairs_ok = rows_ok && T % (2 * kFastBK) == 0 && test_option(GRASS_TEST_NO_PAIRS) == 0;
    if (pairs_ok && planned == kTile256) ks = paired(ks, T);
    const Positions at{pack || (aligned_to(dY0, 16) && ldy0 % 8 == 0 && total % 8 == 0),
                       aligned_to(X, 16) && ldx % 8 == 0 && n % 8 == 0, aligned_to(X, 4)};
    char* base = static_cast<char*>(ws);
    const size_t skip = (256 - reinterpret_cast<uintptr_t>(base) % 256) % 256;
    base += skip;
    TileId tile = kTile128;
    const bool full_f32 = count == 1 && !seg[0].tail && !seg[0].rho && odt == GRASS_F32;
    if (sizes) {
        const Choice c = choose_plan(planned, ks, Shape{T, total, n, layout, gathered, rows_ok, pairs_ok, at, full_f32},
                                     ws_bytes > skip ? ws_bytes - skip : 0);
        tile = c.tile;
        ks = c.k;
    }
    const Copies copy = copies_at(tile, T, total, n, layout, gathered, at);
    pack = pack || copy.a;
    const int64_t nb = copy.b ? (n + 7) / 8 * 8 : n;  // columns the GEMM sees
    // whole aligned 16-byte chunks: what the load-to-LDS kernels and the aligned small tile move
    const bool a_chunks = pack || at.a_chunks;
    const bool aligned = a_chunks && (copy.b || at.x_chunks);
    const bool a_rows_form = rows_ok && tile == kTile256 && aligned;
    const bool a_pairs = a_rows_form && pairs_ok;
    if (a_rows_form) pack = false;
    const Plan p = make_plan(tile, ks, T, total, n, pack);
    uint16_t* panel = reinterpret_cast<uint16_t*>(base);
    float* partial = reinterpret_cast<float*>(base + p.pack_bytes);
    // launch sizes are checked before the first launch: a refused call has done nothing
    const int64_t tiles = static_cast<int64_t>(p.tiles_m) * p.tiles_n;
    const int64_t chunk = (tiles * ks.splits + kNumXcd - 1) / kNumXcd;
    const int64_t blocks = chunk * kNumXcd;
    const int x_chunks = static_cast<int>((nb / 8 + 255) / 256);  // workgroups per row of the aligning copy
    if (blocks > 0x7FFFFFFF || (copy.b && T * x_chunks > 0x7FFFFFFF)) return GRASS_ERR_SHAPE;

    GemmArgs g;
    if (pack) {
        // T x m storage, wide rows: staged through LDS (streaming loads of whole rows)
        // measured on the 60M to 1B layer shapes: from 1024 elements per row on the staged form
        // wins (3 - 15 %), at 512 it loses 20 %; the number of selected rows matters little
        constexpr int64_t min_width = 64, min_m = 1024;
        auto staged = [&](int i, int64_t width) {
            const int64_t m_src = seg[i].src_rows;
            return layout == GRASS_DY_TxM && m_src >= min_m && width >= min_width &&
                   pack_stage_row_elems(m_src) * 2 <= kPackStageMaxBytes;
        };
        auto threads_per_row_log2 = [](int64_t width) {
            int tpr_log2 = 8;  // the power of two covering width / 4
            while (tpr_log2 > 0 && (int64_t{4} << (tpr_log2 - 1)) >= width) --tpr_log2;
            return tpr_log2;
        };
        // several sets, none of them wide: one launch gathers them all
        bool one_launch = count > 1 && layout == GRASS_DY_TxM && T > 0;
        {
            PackSets sets;
            int64_t off = 0, gx = 1, gy = 1;
            for (int i = 0; i < count && one_launch; ++i) {
                const int64_t width = i + 1 == count ? p.rp - off : (seg[i].rows + 7) / 8 * 8;
                if (staged(i, width)) one_launch = false;
                const int tpr_log2 = threads_per_row_log2(width > 0 ? width : 1);
                sets.set[i] = PackSet{static_cast<const uint16_t*>(seg[i].dY), seg[i].ldy, seg[i].idx,
                                      seg[i].rows, width, off, tpr_log2};
                const int64_t rows_per_wg = static_cast<int64_t>(kPackRows) * (256 >> tpr_log2);
                const int64_t bx = (T + rows_per_wg - 1) / rows_per_wg;
                const int64_t by = (width + (int64_t{4} << tpr_log2) - 1) / (int64_t{4} << tpr_log2);
                gx = bx > gx ? bx : gx;
                gy = by > gy ? by : gy;
                off += width;
            }
            if (one_launch) {
                const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(gy),
                                static_cast<unsigned>(count));
                pack_txm_group_kernel<<<grid, 256, 0, s>>>(sets, T, p.rp, panel);
            }
        }
        int64_t off = 0;
        for (int i = 0; i < count && T > 0 && !one_launch; ++i) {
            // the last set also zero-fills the panel's padding columns
            const int64_t width = i + 1 == count ? p.rp - off : (seg[i].rows + 7) / 8 * 8;
            if (width > 0) {
                const int64_t m_src = seg[i].src_rows;  // row length of this set's dY
                if (staged(i, width)) {
                    // wide rows: staged through LDS (streaming loads of whole rows)
                    const auto* src = static_cast<const uint16_t*>(seg[i].dY);
                    const size_t row_bytes = static_cast<size_t>(pack_stage_row_elems(m_src)) * 2;
                    if (m_src < kPackStageDeepMinM)
                        pack_txm_staged_kernel<2, 1><<<static_cast<unsigned>((T + 1) / 2), 256, 2 * row_bytes, s>>>(
                            src, seg[i].ldy, T, m_src, seg[i].idx, seg[i].rows, width, p.rp, panel + off);
                    else if (m_src <= kPackStageTwoRowsMaxM)
                        pack_txm_staged_kernel<2, 4><<<static_cast<unsigned>((T + 1) / 2), 256, 2 * row_bytes, s>>>(
                            src, seg[i].ldy, T, m_src, seg[i].idx, seg[i].rows, width, p.rp, panel + off);
                    else
                        pack_txm_staged_kernel<1, 4><<<static_cast<unsigned>(T), 256, row_bytes, s>>>(
                            src, seg[i].ldy, T, m_src, seg[i].idx, seg[i].rows, width, p.rp, panel + off);
                } else if (layout == GRASS_DY_TxM) {
                    const int tpr_log2 = threads_per_row_log2(width);
                    const int64_t gx = (width + (int64_t{4} << tpr_log2) - 1) / (int64_t{4} << tpr_log2);
                    const int64_t rows_per_wg = static_cast<int64_t>(kPackRows) * (256 >> tpr_log2);
                    const dim3 grid(static_cast<unsigned>((T + rows_per_wg - 1) / rows_per_wg),
                                    static_cast<unsigned>(gx));
                    pack_txm_kernel<<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(seg[i].dY),
                                                         seg[i].ldy, T, seg[i].idx, seg[i].rows,
                                                         width, p.rp, tpr_log2, panel + off);
                } else if (aligned_to(seg[i].dY, 16) && seg[i].ldy % 8 == 0 && p.rp % 8 == 0 &&
                           width % 8 == 0) {
                    const dim3 grid(static_cast<unsigned>((T + kPackWideT - 1) / kPackWideT),
                                    static_cast<unsigned>((width + kPackWideJ - 1) / kPackWideJ));
                    pack_mxt_wide_kernel<<<grid, 256, 0, s>>>(
                        static_cast<const uint16_t*>(seg[i].dY), seg[i].ldy, T, seg[i].idx,
                        seg[i].rows, width, p.rp, panel + off);
                } else {
                    const dim3 grid(static_cast<unsigned>((T + 63) / 64),
                                    static_cast<unsigned>((width + 63) / 64));
                    pack_mxt_kernel<<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(seg[i].dY),
                                                         seg[i].ldy, T, seg[i].idx, seg[i].rows,
                                                         width, p.rp, panel + off);
                }
            }
            off += width;
        }
        g.A = panel;
        g.lda = p.rp;
        g.Mcols = p.rp;
    } else {
        g.A = static_cast<const uint16_t*>(dY0);
        g.lda = ldy0;
        g.Mcols = total;
    }
    g.a_rows = a_rows_form ? seg[0].idx : nullptr;
    g.B = static_cast<const uint16_t*>(X);
    g.ldb = ldx;
    g.Ncols = nb;
    if (copy.b) {
        uint16_t* xa = reinterpret_cast<uint16_t*>(base + p.pack_bytes + round_up(p.partial_bytes, 256));
        align_rows_kernel<<<static_cast<unsigned>(T * x_chunks), 256, 0, s>>>(
            static_cast<const uint16_t*>(X), ldx, T, n, nb, x_chunks, xa);
        g.B = xa;
        g.ldb = nb;
    }
    // a full gradient of one slice is stored where it is wanted: no partial tiles, no pass over them (refresh steps: 6144 x
    // 4096, T = 300: 148 -> 83 us; 5461 x 2048, T = 1000: 108 -> 74, T = 4096: 149 -> 133; 6144 x 6144, T = 4096: 371 -> 335)
    const bool small_staged = tile == kTile128 && !(aligned && sizes);
    bool straight = ks.splits == 1 && full_f32 && !small_staged;
    if (straight) {  // (not over anything that other workgroups still read: the reduction starts when all inputs are used up)
        const Span out = span_of(seg[0].C, total, n, seg[0].ldc, 4);
        straight = !overlap(out, layout == GRASS_DY_MxT ? span_of(dY0, total, T, ldy0, 2) : span_of(dY0, T, total, ldy0, 2)) &&
                   !overlap(out, span_of(X, T, n, ldx, 2)) && !overlap(out, span_of(ws, 1, static_cast<int64_t>(ws_bytes), 0, 1));
    }
    g.P = straight ? static_cast<float*>(seg[0].C) : partial;
    g.K = T;
    g.Mp = p.Mp;
    g.Np = straight ? seg[0].ldc : p.Np;
    g.out_rows = straight ? total : p.Mp;
    g.out_cols = straight ? n : p.Np;
    g.tiles_m = p.tiles_m;
    g.tiles_n = p.tiles_n;
    g.splits = ks.splits;
    // the 128 tile by load-to-LDS where that can fetch the operands (its K tiles are shorter, its sums the same)
    const bool small_direct = tile == kTile128 && aligned && sizes;
    g.ktiles_per_split = static_cast<int>(ks.tokens / (small_direct ? kMidBK : tile_k(tile)));

    const bool a_direct = a_chunks && (test_option(GRASS_TEST_UNALIGNED_X) == 1 ||
                                       (p.tiles_m > 1 && g.ktiles_per_split >= kUnalignedXMin));
    const bool x_direct = !a_chunks && at.x_chunks && !gathered &&
                          (test_option(GRASS_TEST_UNALIGNED_X) == 1 || (p.tiles_n > 1 && g.ktiles_per_split >= kUnalignedXMin));

    const unsigned grid = static_cast<unsigned>(blocks);
    hipError_t le;
    note_kernel(tile == kTileMid ? GRASS_KERNEL_128_256
                : tile == kTile128 ? (small_direct ? GRASS_KERNEL_128 : GRASS_KERNEL_128_STAGED)
                : a_rows_form ? GRASS_KERNEL_256_ROWS
                : aligned ? GRASS_KERNEL_256
                : a_direct ? GRASS_KERNEL_256_UNALIGNED_X
                : x_direct ? GRASS_KERNEL_256_UNALIGNED_DY : GRASS_KERNEL_256_UNALIGNED);
    if (tile == kTile256) {  // the events are stamped with this dispatch's own start and end
        if (a_pairs)
            launch_stamped(tn_gemm_bf16_direct_kernel<false, false, true, true>, dim3(grid), dim3(256), 0, s,
                           ev_start, ev_stop, g);
        else if (a_rows_form)
            launch_stamped(tn_gemm_bf16_direct_kernel<false, false, true>, dim3(grid), dim3(256), 0, s,
                           ev_start, ev_stop, g);
        else if (!aligned && a_direct && gathered)
            launch_stamped(tn_gemm_bf16_unaligned_x_kernel<false>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else if (!aligned && a_direct)
            launch_stamped(tn_gemm_bf16_unaligned_x_kernel<true>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else if (!aligned && x_direct)
            launch_stamped(tn_gemm_bf16_unaligned_x_kernel<true, true>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else if (!aligned && gathered)
            launch_stamped(tn_gemm_bf16_unaligned_kernel<false>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else if (!aligned)
            launch_stamped(tn_gemm_bf16_unaligned_kernel<true>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else if (T % kFastBK != 0 && gathered)
            launch_stamped(tn_gemm_bf16_direct_ragged_kernel<false>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else if (T % kFastBK != 0)
            launch_stamped(tn_gemm_bf16_direct_ragged_kernel<true>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else if (gathered)
            launch_stamped(tn_gemm_bf16_direct_kernel<false>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        else
            launch_stamped(tn_gemm_bf16_direct_kernel<true>, dim3(grid), dim3(256), 0, s, ev_start, ev_stop, g);
        le = hipSuccess;
    } else if (tile == kTileMid) {
        le = raise_lds_limit(reinterpret_cast<const void*>(gathered ? tn_gemm_bf16_mid_kernel<false, 256>
                                                                    : tn_gemm_bf16_mid_kernel<true, 256>),
                             mid_lds_bytes(256), gathered ? 0 : 1);
        if (le == hipSuccess) {
            if (gathered)
                launch_stamped(tn_gemm_bf16_mid_kernel<false, 256>, dim3(grid), dim3(256), mid_lds_bytes(256), s, ev_start, ev_stop, g);
            else
                launch_stamped(tn_gemm_bf16_mid_kernel<true, 256>, dim3(grid), dim3(256), mid_lds_bytes(256), s, ev_start, ev_stop, g);
        }
    } else if (small_direct) {
        if (gathered)
            launch_stamped(tn_gemm_bf16_mid_kernel<false, 128>, dim3(grid), dim3(256), mid_lds_bytes(128), s, ev_start, ev_stop, g);
        else
            launch_stamped(tn_gemm_bf16_mid_kernel<true, 128>, dim3(grid), dim3(256), mid_lds_bytes(128), s, ev_start, ev_stop, g);
        le = hipSuccess;
    } else {
        if (ev_start) (void)hipEventRecord(ev_start, s);
        if (aligned)
            le = gathered ? launch_gemm_kernel<Cfg128, false, false>(g, grid, s)
                          : launch_gemm_kernel<Cfg128, true, false>(g, grid, s);
        else
            le = gathered ? launch_gemm_kernel<Cfg128, false, true>(g, grid, s)
                          : launch_gemm_kernel<Cfg128, true, true>(g, grid, s);
        if (le == hipSuccess && ev_stop) (void)hipEventRecord(ev_stop, s);
    }
    if (le != hipSuccess) return GRASS_ERR_DEVICE;
    if (straight) {
        if (ev_tail_start) (void)hipEventRecord(ev_tail_start, s);
        if (ev_tail_stop) (void)hipEventRecord(ev_tail_stop, s);
        return launch_status();
    }
    return finish_segments(seg, count, partial, ks.splits, p.Mp, p.Np, n, odt, s, ev_tail_start, ev_tail_stop);
}

grass_status launch_tn_gemm(const void* dY, grass_dy_layout layout, int64_t ldy, const void* X,
                            int64_t ldx, grass_dtype dt, int64_t T, int64_t mrows, int64_t n,
                            const int32_t* idx, const float* rho, void* C, grass_dtype odt,
                            int64_t ldc, void* ws, size_t ws_bytes, hipStream_t s,
                            int64_t src_rows, hipEvent_t ev_start, hipEvent_t ev_stop) {
    const GemmSegment one{dY, ldy, idx, rho, C, ldc, mrows, src_rows};
    return launch_tn_gemm_segments(&one, 1, layout, X, ldx, dt, T, n, odt, ws, ws_bytes, s, ev_start, ev_stop);
}

}  // namespace grass
