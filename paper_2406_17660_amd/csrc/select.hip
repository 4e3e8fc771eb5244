// grass_select_rows: compute_P of Section 3.2 on the device.
//
// The work is O(m) integer operations on a few thousand row statistics, so it is latency
// bound, not bandwidth bound: one workgroup of 1024 threads (16 wavefronts) runs the whole
// rule, using LDS histograms, wavefront scans and ballots.  No host round trip: idx and
// rho stay on the device for the calls that follow.
//
//   Top-r           4-pass radix select (8 bits per pass, LDS histogram) on the bit
//                   patterns of sumsq, then an order-preserving compaction by block scan.
//   with repl.      fixed-point weights -> 64-bit inclusive prefix sums in the workspace;
//                   the r draws are independent: Philox word, 64x64 high multiply, binary
//                   search; a per-row hit counter plus a scan emits idx sorted.
//   without repl.   draws are sequential by definition.  Up to 16384 rows, prefix sums over
//                   groups of 64 or 128 rows sit in one wavefront's registers and those of the rows
//                   in LDS (a draw is two compares and one LDS read).  Beyond, a radix-64 sum
//                   tree over the weights (in LDS when it fits in 144 KiB, else in the
//                   workspace) lets the wavefront do a draw in log64(m) steps: 64 children per
//                   load, a wavefront scan and a ballot pick the child; the path is then
//                   decremented.  A scan compacts the chosen rows.
//
// Selection arithmetic is integer, or IEEE double where that gives the same integers (or the
// correctly rounded sqrt / divide), so that the indices are reproducible bit for bit.
#include <atomic>

#include "common.hpp"

// Scratch memory of grass_select_rows_static, the entry point for callers that cannot
// allocate: one copy per GPU, held until the process ends.  In host code this name is only a
// handle for hipGetSymbolAddress; kernels are given the address that call returns.
constexpr size_t kStaticScratchBytes = size_t{1} << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace grass {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr size_t kHeaderBytes = 256;       // status word + padding
constexpr size_t kLdsTreeBytes = 144 * 1024;
constexpr int kMaxLevels = 6;              // 64^6 > 2^31 rows

struct Shared {
    uint32_t hist[256];
    unsigned long long scan_tot[kWaves];
    double red[kWaves];
    unsigned long long bcast64;
    uint32_t prefix;
    uint32_t need;
};

__device__ __forceinline__ uint32_t key_of(float s) { return s == 0.0f ? 0u : __float_as_uint(s); }
__device__ __forceinline__ bool is_bad(float s) { return !(s >= 0.0f) || isinf(s); }

// Philox4x32-10 (Salmon et al., SC'11): counter = (j, refresh_id), key = seed.
__device__ __forceinline__ unsigned long long draw_word(unsigned long long seed,
                                                        unsigned long long refresh,
                                                        unsigned long long j) {
    uint32_t c0 = static_cast<uint32_t>(j), c1 = static_cast<uint32_t>(j >> 32);
    uint32_t c2 = static_cast<uint32_t>(refresh), c3 = static_cast<uint32_t>(refresh >> 32);
    uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        const uint32_t h0 = __umulhi(0xD2511F53u, c0), l0 = 0xD2511F53u * c0;
        const uint32_t h1 = __umulhi(0xCD9E8D57u, c2), l1 = 0xCD9E8D57u * c2;
        const uint32_t n0 = h1 ^ c1 ^ k0, n2 = h0 ^ c3 ^ k1;
        c0 = n0; c1 = l1; c2 = n2; c3 = l0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return static_cast<unsigned long long>(c0) | (static_cast<unsigned long long>(c1) << 32);
}

__device__ __forceinline__ double weight_of(float s, int method) {
    const double d = static_cast<double>(s);
    return method == GRASS_SEL_UNIFORM ? 1.0 : (method == GRASS_SEL_MULTI_NORM ? sqrt(d) : d);
}
__device__ __forceinline__ unsigned long long quantise(double w, double wmax) {
    if (wmax == 0.0) return 1ull;
    return static_cast<unsigned long long>(floor(w / wmax * 1099511627776.0)) + 1ull;
}

// Exclusive prefix sum of one value per thread across the workgroup; `total` is the sum.
// Two barriers; `sh->scan_tot` is reused by every call.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, Shared* sh, T& total) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const T incl = wave_inclusive_scan(v);
    __syncthreads();  // previous users of scan_tot are done
    if (lane == kWave - 1) sh->scan_tot[wave] = static_cast<unsigned long long>(incl);
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const T t = static_cast<T>(sh->scan_tot[w]);
        if (w < wave) before += t;
        all += t;
    }
    total = all;
    return before + incl - v;
}

__device__ __forceinline__ double block_max(double v, Shared* sh) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) sh->red[wave] = v;
    __syncthreads();
    double r = sh->red[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) r = sh->red[w] > r ? sh->red[w] : r;
    return r;
}

// Common prologue: reject NaN / Inf / negative statistics.  `bad`: this thread has seen one.  Returns
// true (for every thread) when any has, after writing the placeholder selection.
__device__ bool report_nonfinite(bool bad, int64_t m, int64_t r, int32_t* idx, float* rho, int32_t* status) {
    if (!__syncthreads_or(bad)) {
        if (threadIdx.x == 0) *status = GRASS_OK;
        return false;
    }
    if (threadIdx.x == 0) *status = GRASS_ERR_NONFINITE;
    for (int64_t j = threadIdx.x; j < r; j += kThreads) {
        idx[j] = static_cast<int32_t>((j * m) / r);  // ascending and inside [0, m)
        rho[j] = 1.0f;
    }
    return true;
}
__device__ bool reject_nonfinite(const float* sumsq, int64_t m, int64_t r, int32_t* idx,
                                 float* rho, int32_t* status) {
    bool bad = false;
    for (int64_t k = threadIdx.x; k < m; k += kThreads) bad |= is_bad(sumsq[k]);
    return report_nonfinite(bad, m, r, idx, rho, status);
}

// Up to 16384 rows (every layer's row count in practice) each thread keeps PER consecutive rows in
// registers: the statistic is read once, with all loads in flight, and a compaction needs a single
// block scan, where the kernels for any size read it in up to six passes of m / 1024 dependent
// rounds and scan once per round.  Those rounds are what the small selections spend their time on
// (13824 rows: Top-r 36 -> 29 us, with replacement 65 -> 31 us; 4096 rows: 12.6 -> 11.3
// and 25 -> 16 us).
constexpr int kRegRows = 16;
constexpr int64_t kRegMaxRows = int64_t{kRegRows} * kThreads;
template <int PER>
__device__ __forceinline__ bool load_rows(const float* sumsq, int m, int first, int count, float (&s)[PER]) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < PER; ++i) s[i] = i < count && first + i < m ? sumsq[first + i] : 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) bad |= is_bad(s[i]);
    return bad;
}

// ------------------------------------------------------------------------------ Top-r
// One pass of the radix select, by one wavefront: the digit at which the count of rows with a larger
// digit first reaches `need`.  Lane L owns digits 255-4L .. 252-4L (descending).
__device__ __forceinline__ void find_digit(Shared* sh, uint32_t prefix, uint32_t need, int shift) {
    const int lane = threadIdx.x;
    uint32_t h[4], s = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) { h[e] = sh->hist[255 - 4 * lane - e]; s += h[e]; }
    const uint32_t incl = wave_inclusive_scan(s);
    uint32_t above = incl - s;
    if (above < need && need <= incl) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (need <= above + h[e]) {
                sh->prefix = prefix | (static_cast<uint32_t>(255 - 4 * lane - e) << shift);
                sh->need = need - above;
                break;
            }
            above += h[e];
        }
    }
}

// The rows in registers (see load_rows); otherwise the kernel below.
template <int PER>
__global__ __launch_bounds__(kThreads) void select_topr_reg_kernel(
    const float* __restrict__ sumsq, int m, int r, int32_t* __restrict__ idx, float* __restrict__ rho,
    int32_t* __restrict__ status) {
    __shared__ Shared sh;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int per = (m + kThreads - 1) / kThreads, first = tid * per;
    float s[PER];
    const bool bad = load_rows(sumsq, m, first, per, s);
    if (report_nonfinite(bad, m, r, idx, rho, status)) return;
    if (r == 0) return;  // nothing to select: only the status word is written
    const int mine = first >= m ? 0 : (m - first < per ? m - first : per);  // rows of this thread

    uint32_t prefix = 0, need = static_cast<uint32_t>(r);
    for (int pass = 3; pass >= 0; --pass) {
        const int shift = pass * 8;
        if (tid < 256) sh.hist[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (i >= per) continue;
            const uint32_t key = key_of(s[i]), digit = (key >> shift) & 255u;
            bool count = i < mine && (pass == 3 || (key >> (shift + 8)) == (prefix >> (shift + 8)));
            // the leading digits are nearly all alike (sign and exponent): one add per value and
            // wavefront instead of 64 that would queue for one LDS word
            for (int round = 0; pass == 3 && round < 4; ++round) {
                const unsigned long long left = __ballot(count);
                if (!left) break;
                const int leader = __ffsll(static_cast<long long>(left)) - 1;
                const bool same = count && digit == static_cast<uint32_t>(__builtin_amdgcn_readlane(digit, leader));
                const int n = __popcll(__ballot(same));
                if (lane == leader) atomicAdd(&sh.hist[digit], static_cast<uint32_t>(n));
                count = count && !same;
            }
            if (count) atomicAdd(&sh.hist[digit], 1u);
        }
        __syncthreads();
        if (tid < kWave) find_digit(&sh, prefix, need, shift);
        __syncthreads();
        prefix = sh.prefix;
        need = sh.need;
    }

    // every key above the threshold, and the first `need` rows that equal it (ties go to the
    // lower index), in row order; low 32 bits: rows above, high: rows equal
    unsigned long long counts = 0, total;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t key = key_of(s[i]);
        if (i < mine) counts += (key > prefix ? 1ull : 0ull) | (key == prefix ? (1ull << 32) : 0ull);
    }
    const unsigned long long before = block_exclusive_scan(counts, &sh, total);
    uint32_t gt = static_cast<uint32_t>(before), eq = static_cast<uint32_t>(before >> 32);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (i >= mine) continue;
        const uint32_t key = key_of(s[i]);
        if (key > prefix || (key == prefix && eq < need)) {
            const uint32_t pos = gt + (eq < need ? eq : need);
            idx[pos] = first + i;
            rho[pos] = 1.0f;
        }
        gt += key > prefix;
        eq += key == prefix;
    }
}

__global__ __launch_bounds__(kThreads) void select_topr_kernel(
    const float* __restrict__ sumsq, int64_t m, int64_t r, int32_t* __restrict__ idx,
    float* __restrict__ rho, int32_t* __restrict__ status) {
    __shared__ Shared sh;
    if (reject_nonfinite(sumsq, m, r, idx, rho, status)) return;
    if (r == 0) return;  // nothing to select: only the status word is written
    const int tid = threadIdx.x;

    // Radix select: after the four passes `prefix` is the r-th largest key and `need`
    // how many rows carrying exactly that key are still wanted.
    uint32_t prefix = 0, need = static_cast<uint32_t>(r);
    for (int pass = 3; pass >= 0; --pass) {
        const int shift = pass * 8;
        if (tid < 256) sh.hist[tid] = 0;
        __syncthreads();
        for (int64_t k = tid; k < m; k += kThreads) {
            const uint32_t key = key_of(sumsq[k]);
            const bool match = pass == 3 || (key >> (shift + 8)) == (prefix >> (shift + 8));
            if (match) atomicAdd(&sh.hist[(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (tid < kWave) find_digit(&sh, prefix, need, shift);
        __syncthreads();
        prefix = sh.prefix;
        need = sh.need;
    }

    // Compaction in row order: every key above the threshold, and the first `need` rows
    // that equal it (ties go to the lower index).
    unsigned long long carry = 0;  // low 32 bits: rows above so far; high: rows equal so far
    for (int64_t base = 0; base < m; base += kThreads) {
        const int64_t k = base + tid;
        bool gt = false, eq = false;
        if (k < m) {
            const uint32_t key = key_of(sumsq[k]);
            gt = key > prefix;
            eq = key == prefix;
        }
        const unsigned long long mine = (gt ? 1ull : 0ull) | (eq ? (1ull << 32) : 0ull);
        unsigned long long total;
        const unsigned long long before = carry + block_exclusive_scan(mine, &sh, total);
        const uint32_t gt_before = static_cast<uint32_t>(before);
        const uint32_t eq_before = static_cast<uint32_t>(before >> 32);
        if (gt || (eq && eq_before < need)) {
            const uint32_t pos = gt_before + (eq_before < need ? eq_before : need);
            idx[pos] = static_cast<int32_t>(k);
            rho[pos] = 1.0f;
        }
        carry += total;
    }
}

// ------------------------------------------------------------------------------ with replacement
__global__ __launch_bounds__(kThreads) void select_repl_kernel(
    const float* __restrict__ sumsq, int64_t m, int64_t r, int method, int rescale,
    unsigned long long seed, unsigned long long refresh, int32_t* __restrict__ idx,
    float* __restrict__ rho, int32_t* __restrict__ status, unsigned long long* __restrict__ csum,
    uint32_t* __restrict__ hits) {
    __shared__ Shared sh;
    if (reject_nonfinite(sumsq, m, r, idx, rho, status)) return;
    if (r == 0) return;  // nothing to select: only the status word is written
    const int tid = threadIdx.x;

    double wmax = 0.0;
    for (int64_t k = tid; k < m; k += kThreads) {
        const double w = weight_of(sumsq[k], method);
        wmax = w > wmax ? w : wmax;
    }
    wmax = block_max(wmax, &sh);

    // inclusive prefix sums of the integer weights
    unsigned long long carry = 0;
    for (int64_t base = 0; base < m; base += kThreads) {
        const int64_t k = base + tid;
        const unsigned long long wq = k < m ? quantise(weight_of(sumsq[k], method), wmax) : 0ull;
        unsigned long long total;
        const unsigned long long before = block_exclusive_scan(wq, &sh, total);
        if (k < m) {
            csum[k] = carry + before + wq;
            hits[k] = 0;
        }
        carry += total;
    }
    const unsigned long long total_w = carry;
    __threadfence_block();
    __syncthreads();

    // independent draws: first k with csum[k] > target
    for (int64_t j = tid; j < r; j += kThreads) {
        const unsigned long long target = __umul64hi(draw_word(seed, refresh, j), total_w);
        int64_t lo = 0, hi = m - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (csum[mid] > target) hi = mid; else lo = mid + 1;
        }
        atomicAdd(&hits[lo], 1u);
    }
    __threadfence_block();
    __syncthreads();

    // emit rows in ascending order, each as often as it was hit
    uint32_t out_carry = 0;
    for (int64_t base = 0; base < m; base += kThreads) {
        const int64_t k = base + tid;
        const uint32_t h = k < m ? hits[k] : 0u;
        uint32_t total;
        const uint32_t pos = out_carry + block_exclusive_scan(h, &sh, total);
        if (h) {
            float rk = 1.0f;
            if (rescale) {
                const unsigned long long wq = csum[k] - (k ? csum[k - 1] : 0ull);
                const double q = static_cast<double>(wq) / static_cast<double>(total_w);
                rk = static_cast<float>(1.0 / sqrt(static_cast<double>(r) * q));
            }
            for (uint32_t e = 0; e < h; ++e) {
                idx[pos + e] = static_cast<int32_t>(k);
                rho[pos + e] = rk;
            }
        }
        out_carry += total;
    }
}

// The rows in registers (see load_rows) and the prefix sums in LDS, where the draws' binary searches
// run; otherwise the kernel above.
template <int PER>
__global__ __launch_bounds__(kThreads) void select_repl_reg_kernel(
    const float* __restrict__ sumsq, int m, int64_t r, int method, int rescale, unsigned long long seed,
    unsigned long long refresh, int32_t* __restrict__ idx, float* __restrict__ rho,
    int32_t* __restrict__ status, uint32_t* __restrict__ ws_hits) {
    __shared__ Shared sh;
    // m inclusive prefix sums of the integer weights, then, while both fit in 48 KB, the m hit counters
    extern __shared__ unsigned long long lds_csum[];
    uint32_t* hits = PER < kRegRows ? reinterpret_cast<uint32_t*>(lds_csum + m) : ws_hits;
    const int tid = threadIdx.x;
    const int per = (m + kThreads - 1) / kThreads, first = tid * per;
    float s[PER], smax = 0.f;
    const bool bad = load_rows(sumsq, m, first, per, s);
    if (report_nonfinite(bad, m, r, idx, rho, status)) return;
    if (r == 0) return;  // nothing to select: only the status word is written
    const int mine = first >= m ? 0 : (m - first < per ? m - first : per);  // rows of this thread
    // the weights are monotone in the statistic: the largest weight is that of the largest one
#pragma unroll
    for (int i = 0; i < PER; ++i) smax = s[i] > smax ? s[i] : smax;
    const double wmax = weight_of(static_cast<float>(block_max(static_cast<double>(smax), &sh)), method);
    unsigned long long wq[PER], sum = 0, total_w;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        wq[i] = 0;
        if (i < mine) {
            wq[i] = quantise(weight_of(s[i], method), wmax);
            hits[first + i] = 0;
        }
        sum += wq[i];
    }
    unsigned long long run = block_exclusive_scan(sum, &sh, total_w);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        run += wq[i];
        if (i < mine) lds_csum[first + i] = run;
    }
    __threadfence_block();
    __syncthreads();

    // independent draws: first k with csum[k] > target
    for (int64_t j = tid; j < r; j += kThreads) {
        const unsigned long long target = __umul64hi(draw_word(seed, refresh, j), total_w);
        int lo = 0, hi = m - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (lds_csum[mid] > target) hi = mid; else lo = mid + 1;
        }
        atomicAdd(&hits[lo], 1u);
    }
    __threadfence_block();
    __syncthreads();

    // emit rows in ascending order, each as often as it was hit
    uint32_t h[PER], count = 0, all;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        h[i] = i < mine ? hits[first + i] : 0u;
        count += h[i];
    }
    uint32_t pos = block_exclusive_scan(count, &sh, all);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (h[i] == 0) continue;
        float rk = 1.0f;
        if (rescale) {
            const double q = static_cast<double>(wq[i]) / static_cast<double>(total_w);
            rk = static_cast<float>(1.0 / sqrt(static_cast<double>(r) * q));
        }
        for (uint32_t e = 0; e < h[i]; ++e) {
            idx[pos + e] = first + i;
            rho[pos + e] = rk;
        }
        pos += h[i];
    }
}

// ------------------------------------------------------------------------------ without replacement
// Sampling without replacement is r sequential draws from the weights that are left (the
// weight of a drawn row is taken out before the next draw).  The weights sit in a radix-64
// tree whose nodes store, instead of their own sum, the INCLUSIVE PREFIX of the sums inside
// their group of 64 siblings.  One wavefront then walks a draw down the tree with one load,
// one compare and one ballot per level (the first lane whose prefix exceeds the target is
// the child to enter; the prefix of the lane before it is what the target loses), and takes
// the drawn weight w out by subtracting w from the prefixes at and after the path's lane in
// each of the path's groups.  Every value is an exact integer, so the draws are those of the
// sequential definition.  Every level is padded to whole groups; padding carries weight 0.
struct TreeShape {
    int levels;                  // level 0 = leaves
    int64_t groups[kMaxLevels];  // groups of 64 entries per level (the top level has one)
    int64_t offset[kMaxLevels];  // first entry of the level inside the node array
};

__device__ __forceinline__ unsigned long long read_lane64(unsigned long long v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(v), l);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(v >> 32), l);
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// The r draws, by one wavefront.  TreePtr is an LDS or a global pointer; kFence orders the
// updates of a global tree before the next draw's loads.
template <int LEVELS, bool kFence, typename TreePtr>
__device__ __forceinline__ void draw_without_replacement(TreePtr tree, const TreeShape& shape,
                                                         int64_t r, unsigned long long seed,
                                                         unsigned long long refresh,
                                                         unsigned long long total_w, int lane) {
    unsigned long long remaining = total_w;
    for (int64_t j0 = 0; j0 < r; j0 += kWave) {
        // the Philox words of the next 64 draws, one per lane
        const unsigned long long words = draw_word(seed, refresh, static_cast<unsigned long long>(j0 + lane));
        const int in_block = r - j0 < kWave ? static_cast<int>(r - j0) : kWave;
        for (int jj = 0; jj < in_block; ++jj) {
            unsigned long long target = __umul64hi(read_lane64(words, jj), remaining);
            unsigned long long prefix[LEVELS];
            int64_t entry[LEVELS];
            int first[LEVELS];
            unsigned long long w = 0;
            int64_t node = 0;
#pragma unroll
            for (int L = LEVELS - 1; L >= 0; --L) {
                entry[L] = shape.offset[L] + node * kWave + lane;
                prefix[L] = tree[entry[L]];
                const unsigned long long hit = __ballot(prefix[L] > target);
                const int f = __ffsll(static_cast<long long>(hit)) - 1;  // hit != 0: target < total
                const unsigned long long before = f > 0 ? read_lane64(prefix[L], f - 1) : 0ull;
                if (L == 0) w = read_lane64(prefix[0], f) - before;  // the leaf drawn
                target -= before;
                first[L] = f;
                node = node * kWave + f;
            }
#pragma unroll
            for (int L = 0; L < LEVELS; ++L)
                if (lane >= first[L]) tree[entry[L]] = prefix[L] - w;
            remaining -= w;
            if (kFence) __threadfence_block();
        }
    }
}

template <bool kFence, typename TreePtr>
__device__ __forceinline__ void draw_dispatch(TreePtr tree, const TreeShape& shape, int64_t r,
                                              unsigned long long seed, unsigned long long refresh,
                                              unsigned long long total_w, int lane) {
    switch (shape.levels) {
        case 1: draw_without_replacement<1, kFence>(tree, shape, r, seed, refresh, total_w, lane); break;
        case 2: draw_without_replacement<2, kFence>(tree, shape, r, seed, refresh, total_w, lane); break;
        case 3: draw_without_replacement<3, kFence>(tree, shape, r, seed, refresh, total_w, lane); break;
        case 4: draw_without_replacement<4, kFence>(tree, shape, r, seed, refresh, total_w, lane); break;
        case 5: draw_without_replacement<5, kFence>(tree, shape, r, seed, refresh, total_w, lane); break;
        default: draw_without_replacement<6, kFence>(tree, shape, r, seed, refresh, total_w, lane); break;
    }
}

template <bool kTreeInLds>
__global__ __launch_bounds__(kThreads) void select_norepl_kernel(
    const float* __restrict__ sumsq, int64_t m, int64_t r, int method, int rescale,
    unsigned long long seed, unsigned long long refresh, int32_t* __restrict__ idx,
    float* __restrict__ rho, int32_t* __restrict__ status, unsigned long long* ws_tree,
    TreeShape shape) {
    __shared__ Shared sh;
    extern __shared__ unsigned long long lds_tree[];
    if (reject_nonfinite(sumsq, m, r, idx, rho, status)) return;
    if (r == 0) return;  // nothing to select: only the status word is written
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    unsigned long long* tree = kTreeInLds ? lds_tree : ws_tree;

    double wmax = 0.0;
    for (int64_t k = tid; k < m; k += kThreads) {
        const double w = weight_of(sumsq[k], method);
        wmax = w > wmax ? w : wmax;
    }
    wmax = block_max(wmax, &sh);

    // padding entries of the inner levels (children that do not exist) weigh 0
    for (int L = 1; L < shape.levels; ++L)
        for (int64_t e = shape.groups[L - 1] + tid; e < shape.groups[L] * kWave; e += kThreads)
            tree[shape.offset[L] + e] = 0ull;
    __threadfence_block();
    __syncthreads();
    // level by level: prefix sums inside each group; the group's sum goes up one level
    for (int L = 0; L < shape.levels; ++L) {
        for (int64_t g = wave; g < shape.groups[L]; g += kWaves) {
            const int64_t e = g * kWave + lane;
            unsigned long long v;
            if (L == 0) v = e < m ? quantise(weight_of(sumsq[e], method), wmax) : 0ull;
            else v = tree[shape.offset[L] + e];
            v = wave_inclusive_scan(v);
            tree[shape.offset[L] + e] = v;
            if (lane == kWave - 1 && L + 1 < shape.levels) tree[shape.offset[L + 1] + g] = v;
        }
        __threadfence_block();
        __syncthreads();
    }
    const unsigned long long total_w = tree[shape.offset[shape.levels - 1] + kWave - 1];

    if (wave == 0) draw_dispatch<!kTreeInLds>(tree, shape, r, seed, refresh, total_w, lane);
    __threadfence_block();
    __syncthreads();

    // chosen leaves now weigh 0 (every weight started >= 1): compact them in row order
    uint32_t carry = 0;
    for (int64_t base = 0; base < m; base += kThreads) {
        const int64_t k = base + tid;
        uint32_t chosen = 0;
        if (k < m) {
            const unsigned long long here = tree[k];  // level 0 starts at offset 0
            const unsigned long long before = (k & (kWave - 1)) ? tree[k - 1] : 0ull;
            chosen = here == before ? 1u : 0u;
        }
        uint32_t total;
        const uint32_t pos = carry + block_exclusive_scan(chosen, &sh, total);
        if (chosen) {
            float rk = 1.0f;
            if (rescale) {
                const unsigned long long wq = quantise(weight_of(sumsq[k], method), wmax);
                const double q = static_cast<double>(wq) / static_cast<double>(total_w);
                rk = static_cast<float>(1.0 / sqrt(static_cast<double>(r) * q));
            }
            idx[pos] = static_cast<int32_t>(k);
            rho[pos] = rk;
        }
        carry += total;
    }
}

// The same draws for up to 16384 rows with fewer instructions from one draw to the next.  What
// bounds sampling without replacement is that chain: draw j needs the weight that draw j - 1 took
// out, one wavefront runs it, and a lone wavefront issues an instruction every five to eight clocks.
// The tree above spends an LDS round trip, a ballot and an update per level (three levels at
// m = 13824: 0.40 us per draw).  Here the weights of 64 R rows form a group whose inclusive prefix sums
// lie in LDS (R consecutive rows per lane), and the EXCLUSIVE prefix sums over the groups (at most 64 E)
// stay in E registers per lane:
//   group   g = (number of groups whose prefix is <= target) - 1: E compares and bit counts
//   row     f = number of rows of the group whose prefix is <= target - prefix(g): R of each
//   weight  difference of neighbouring prefixes, formed by a lane shift
//   update  the lanes that failed a compare are the ones that lose the weight
// and the drawn rows are collected in a register and put into a bit map 64 at a time.
//
// While the total weight is below 2^53 (always for fewer than 8192 rows, and for more unless most
// weigh as much as the heaviest) every prefix and difference is an integer that a double holds
// exactly, and the fifteen instructions of the high product become a single double one.  Only the target x S / 2^64 is rounded: the double product
// is within 2 of it, so unless a prefix lies within 4 (checked against every prefix compared) each
// comparison falls as with the exact target floor(x S / 2^64); otherwise that is computed and used.
// The rows drawn are those of the sequential integer definition in every case.  From 2^53 on (uniform weights of 8192
// rows and more) the same draw runs in 64-bit integers: 220 us for 1100 of 8801 rows, 402 for 2048 of 13720; in a
// loop of its own, with selects instead of masks and one draw a turn, 321 and 591.
// E, R = 1, 1 up to 4096 rows, 1, 2 up to 8192 and 2, 2 up to 16384.  1024 draws take 128 us of 4096 rows,
// 153 of 8192 and 177 of 13824; before the masks went into EXEC, four draws into a turn of the loop, the
// weight ahead of the updates and two rows into a lane: 166, 188 and 264 (E, R = 1, 1; 2, 1; 4, 1), with the
// three-level tree 286 of 4096 and 420 of 13824.  E, R = 2, 1 of 8192 rows and 4, 1 of 13824 in the present
// form: 153 and 204.  (Guessing the next draw's group a draw ahead, to hide the one LDS read, costs more
// instructions than the read takes; forming the next target in every lane before the drawn one is known
// saves a multiplication and costs two reads of a lane: 160 against 153.)
constexpr int64_t kFlatMaxRows = int64_t{4} * kWave * kWave;

// v of the lane below, 0 in lane 0
__device__ __forceinline__ unsigned long long from_lane_below(unsigned long long v) {
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x138, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), 0x138, 0xf, 0xf, true);
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

__device__ __forceinline__ double from_lane_below(double v) {
    return __longlong_as_double(static_cast<long long>(from_lane_below(static_cast<unsigned long long>(__double_as_longlong(v)))));
}
__device__ __forceinline__ unsigned long long read_lane(unsigned long long v, int l) { return read_lane64(v, l); }
__device__ __forceinline__ double read_lane(double v, int l) {
    return __longlong_as_double(static_cast<long long>(read_lane64(static_cast<unsigned long long>(__double_as_longlong(v)), l)));
}

// lane l of v becomes x (both the same for the whole wavefront)
__device__ __forceinline__ void write_lane(int& v, int x, int l) {
    asm("s_mov_b32 m0, %2\n\tv_writelane_b32 %0, %1, m0" : "+v"(v) : "s"(x), "s"(l) : "m0");
}

// A draw, in doubles or in 64-bit integers.  pex[e]: the weight before group E * lane + e (more than any target for
// groups that do not exist).  near (doubles): some boundary of the group lies within 4 of the target, the only
// ones a target off by 2 could be on the wrong side of (a target put into the wrong group is next to that group's edge).
template <typename V, int E, int R>
struct Draw {
    int n, f;  // group n - 1, row f of it
    V cur[R], w;
    unsigned long long upto[E], below[R];  // the lanes outside these masks lose the drawn weight
    bool near;
};
template <typename V, int E, int R>
__device__ __forceinline__ Draw<V, E, R> locate(const V (&pex)[E], const V* leaf, V target, int lane) {
    constexpr bool kRounded = static_cast<V>(0.5) != static_cast<V>(0);
    Draw<V, E, R> q;
    q.n = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        q.upto[e] = __ballot(pex[e] <= target);
        q.n += __popcll(q.upto[e]);  // at least 1: the first group's prefix is 0
    }
    const V* src = leaf + (lane - kWave) * R + q.n * (kWave * R);
#pragma unroll
    for (int i = 0; i < R; ++i) q.cur[i] = src[i];
    V before = pex[0];  // of the last of this lane's groups that starts at or before the target
#pragma unroll
    for (int e = 1; e < E; ++e) before = pex[e] <= target ? pex[e] : before;
    before = read_lane(before, (__popcll(q.upto[0]) - 1) & (kWave - 1));
    __builtin_amdgcn_sched_barrier(0);  // while the read is under way: nothing that waits for it moves up
    V own = q.cur[0] - from_lane_below(q.cur[R - 1]);
    const V t = target - before;
    V least = t;
    q.f = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        q.below[i] = __ballot(q.cur[i] <= t);
        q.f += __popcll(q.below[i]);
        if (i > 0) own = q.cur[i - 1] <= t ? q.cur[i] - q.cur[i - 1] : own;
        if constexpr (kRounded) least = fmin(fabs(q.cur[i] - t), least);
    }
    if constexpr (kRounded) q.near = __ballot(least < 4.0) != 0;
    else q.near = false;
    q.w = read_lane(own, __popcll(q.below[R - 1]) & (kWave - 1));  // the first lane with a row past the target
    return q;
}
// Takes w out of the drawn row's group (the row and those after it) and of the groups after its own.  All
// 64 lanes are active before and after: with a mask in EXEC a subtraction is one vector instruction
// instead of three (two selects and an addition).  The s_nop: w may come from the instruction just before,
// a v_readlane, and a vector instruction may read a scalar register two wait states after one wrote it.
#define GRASS_SUB_F64(d, w) "v_add_f64 " d ", " d ", -" w "\n\t"
#define GRASS_SUB_U64(d, w) "v_lshl_add_u64 " d ", " d ", 0, " w "\n\t"  // w: its negative
#define GRASS_TAKE_OUT(SUB, W)                                                                                       \
    if constexpr (R == 1)                                                                                            \
        asm("s_not_b64 exec, %3\n\ts_nop 0\n\t" SUB("%0", "%2") "s_not_b64 exec, %4\n\t" SUB("%1", "%2")             \
            "s_mov_b64 exec, -1"                                                                                     \
            : "+v"(pex[0]), "+v"(q.cur[0]) : "s"(W), "s"(q.upto[0]), "s"(q.below[0]) : "scc");                       \
    else if constexpr (E == 1)                                                                                       \
        asm("s_not_b64 exec, %4\n\ts_nop 0\n\t" SUB("%0", "%3") "s_not_b64 exec, %5\n\t" SUB("%1", "%3")             \
            "s_not_b64 exec, %6\n\t" SUB("%2", "%3") "s_mov_b64 exec, -1"                                            \
            : "+v"(pex[0]), "+v"(q.cur[0]), "+v"(q.cur[1])                                                           \
            : "s"(W), "s"(q.upto[0]), "s"(q.below[0]), "s"(q.below[1]) : "scc");                                     \
    else                                                                                                             \
        asm("s_not_b64 exec, %5\n\ts_nop 0\n\t" SUB("%0", "%4") "s_not_b64 exec, %6\n\t" SUB("%1", "%4")             \
            "s_not_b64 exec, %7\n\t" SUB("%2", "%4") "s_not_b64 exec, %8\n\t" SUB("%3", "%4") "s_mov_b64 exec, -1"   \
            : "+v"(pex[0]), "+v"(pex[E - 1]), "+v"(q.cur[0]), "+v"(q.cur[R - 1])                                     \
            : "s"(W), "s"(q.upto[0]), "s"(q.upto[E - 1]), "s"(q.below[0]), "s"(q.below[R - 1]) : "scc")
template <typename V, int E, int R>
__device__ __forceinline__ void take_out(Draw<V, E, R>& q, V (&pex)[E], V* leaf, int lane) {
    static_assert(E <= R && R <= 2, "the forms above");
    if constexpr (static_cast<V>(0.5) != static_cast<V>(0)) {
        GRASS_TAKE_OUT(GRASS_SUB_F64, q.w);
    } else {
        const V minus = 0 - q.w;
        GRASS_TAKE_OUT(GRASS_SUB_U64, minus);
    }
    V* dst = leaf + (lane - kWave) * R + q.n * (kWave * R);
#pragma unroll
    for (int i = 0; i < R; ++i) dst[i] = q.cur[i];
}
#undef GRASS_TAKE_OUT
#undef GRASS_SUB_U64
#undef GRASS_SUB_F64

template <int E, int R>
__global__ __launch_bounds__(kThreads) void select_norepl_flat_kernel(
    const float* __restrict__ sumsq, int m, int r, int method, int rescale, unsigned long long seed,
    unsigned long long refresh, int32_t* __restrict__ idx, float* __restrict__ rho,
    int32_t* __restrict__ status) {
    constexpr int kGroupsPerWave = E * kWave / kWaves;
    __shared__ Shared sh;
    __shared__ unsigned long long gsum[E * kWave];
    constexpr int kWords = E * R * kWave * 2;
    __shared__ uint32_t chosen[kWords];  // one bit per row
    extern __shared__ __attribute__((aligned(16))) unsigned long long leaf[];  // [groups][64 R] inclusive prefix sums, or their doubles
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int groups = (m + kWave * R - 1) / (kWave * R);

    float s[kGroupsPerWave][R], smax = 0.f;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < kGroupsPerWave; ++i)
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int k = ((wave + i * kWaves) * kWave + lane) * R + u;
            s[i][u] = k < m ? sumsq[k] : 0.f;
        }
#pragma unroll
    for (int i = 0; i < kGroupsPerWave; ++i)
#pragma unroll
        for (int u = 0; u < R; ++u) {
            bad |= is_bad(s[i][u]);
            smax = s[i][u] > smax ? s[i][u] : smax;
        }
    if (report_nonfinite(bad, m, r, idx, rho, status)) return;
    if (r == 0) return;  // nothing to select: only the status word is written
    // the weights are monotone in the statistic: the largest weight is that of the largest one
    const double wmax = weight_of(static_cast<float>(block_max(static_cast<double>(smax), &sh)), method);
    unsigned long long prefix[kGroupsPerWave][R];
#pragma unroll
    for (int i = 0; i < kGroupsPerWave; ++i) {
        const int g = wave + i * kWaves;
        if (g < groups) {  // (the same for the whole wavefront)
            unsigned long long sum = 0;
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int k = (g * kWave + lane) * R + u;
                sum += k < m ? quantise(weight_of(s[i][u], method), wmax) : 0ull;
                prefix[i][u] = sum;
            }
            const unsigned long long before = wave_inclusive_scan(sum) - sum;
#pragma unroll
            for (int u = 0; u < R; ++u) prefix[i][u] += before;
        } else {  // groups that do not exist weigh nothing
#pragma unroll
            for (int u = 0; u < R; ++u) prefix[i][u] = 0ull;
        }
        if (lane == kWave - 1) gsum[g] = prefix[i][R - 1];
    }
    for (int e = tid; e < kWords; e += kThreads) chosen[e] = 0;
    __syncthreads();
    unsigned long long pex[E], total_w;  // pex[e]: weight before group E * lane + e
    {
        unsigned long long own[E], lane_sum = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            own[e] = gsum[E * lane + e];
            lane_sum += own[e];
        }
        const unsigned long long incl = wave_inclusive_scan(lane_sum);
        total_w = read_lane64(incl, kWave - 1);
        pex[0] = incl - lane_sum;
#pragma unroll
        for (int e = 1; e < E; ++e) pex[e] = pex[e - 1] + own[e - 1];
    }
    const bool in_doubles = total_w < (1ull << 53);
#pragma unroll
    for (int i = 0; i < kGroupsPerWave; ++i) {
        const int g = wave + i * kWaves;
        if (g < groups)
#pragma unroll
            for (int u = 0; u < R; ++u)
                leaf[(g * kWave + lane) * R + u] = in_doubles
                    ? static_cast<unsigned long long>(__double_as_longlong(static_cast<double>(prefix[i][u]))) : prefix[i][u];
    }
    __syncthreads();

    if (wave == 0) {
        double* dleaf = reinterpret_cast<double*>(leaf);
        double dpex[E], dleft = static_cast<double>(total_w);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            dpex[e] = E * lane + e < groups ? static_cast<double>(pex[e]) : __builtin_inf();
            if (E * lane + e >= groups) pex[e] = ~0ull;  // (stays above every target: it loses at most the total)
        }
        unsigned long long left = total_w;
        for (int j0 = 0; j0 < r; j0 += kWave) {
            const unsigned long long words = draw_word(seed, refresh, j0 + lane);
            const double unit = static_cast<double>(words) * 0x1p-64;
            const int count = __builtin_amdgcn_readfirstlane(r - j0 < kWave ? r - j0 : kWave);
            int rows = 0;  // lane jj: the row of draw j0 + jj
            auto four_a_turn = [&](auto draw) {  // a taken branch costs a lone wavefront tens of clocks
                int jj = 0;
                for (; jj + 4 <= count; jj += 4) {
                    draw(jj);
                    draw(jj + 1);
                    draw(jj + 2);
                    draw(jj + 3);
                }
                for (; jj < count; ++jj) draw(jj);
            };
            if (in_doubles) {
                double target = dleft * read_lane(unit, 0);
                four_a_turn([&](int jj) {
                    const double next_unit = read_lane(unit, (jj + 1) & (kWave - 1));
                    auto q = locate<double, E, R>(dpex, dleaf, target, lane);
                    if (__builtin_expect(q.near, 0)) {  // too close to a boundary to call: the exact target
                        const unsigned long long exact =
                            __umul64hi(read_lane64(words, jj), static_cast<unsigned long long>(dleft));
                        q = locate<double, E, R>(dpex, dleaf, static_cast<double>(exact), lane);
                    }
                    // the next draw's target first: it is what the next draw begins with
                    dleft -= q.w;
                    target = dleft * next_unit;
                    take_out<double, E, R>(q, dpex, dleaf, lane);
                    write_lane(rows, (q.n - 1) * (kWave * R) + q.f, jj);
                });
            } else {
                unsigned long long target = __umul64hi(read_lane64(words, 0), left);
                four_a_turn([&](int jj) {
                    const unsigned long long next_word = read_lane64(words, (jj + 1) & (kWave - 1));
                    auto q = locate<unsigned long long, E, R>(pex, leaf, target, lane);
                    left -= q.w;
                    target = __umul64hi(next_word, left);
                    take_out<unsigned long long, E, R>(q, pex, leaf, lane);
                    write_lane(rows, (q.n - 1) * (kWave * R) + q.f, jj);
                });
            }
            if (lane < count) atomicOr(&chosen[rows >> 5], 1u << (rows & 31));
        }
    }
    __syncthreads();

    // emit the chosen rows in ascending order: every thread owns 32 consecutive rows
    static_assert(kWords <= kThreads, "one word of the bit map per thread");
    uint32_t bits = tid < kWords ? chosen[tid] : 0u, all;
    uint32_t pos = block_exclusive_scan(static_cast<uint32_t>(__popc(bits)), &sh, all);
    while (bits) {
        const int k = tid * 32 + __ffs(bits) - 1;
        bits &= bits - 1;
        float rk = 1.0f;
        if (rescale) {
            const unsigned long long wq = quantise(weight_of(sumsq[k], method), wmax);
            const double q = static_cast<double>(wq) / static_cast<double>(total_w);
            rk = static_cast<float>(1.0 / sqrt(static_cast<double>(r) * q));
        }
        idx[pos] = k;
        rho[pos] = rk;
        ++pos;
    }
}

TreeShape tree_shape(int64_t m) {
    TreeShape s;
    s.levels = 0;
    int64_t groups = m > 0 ? (m + kWave - 1) / kWave : 1, off = 0;
    while (true) {
        s.groups[s.levels] = groups;
        s.offset[s.levels] = off;
        ++s.levels;
        if (groups == 1 || s.levels == kMaxLevels) break;
        off += groups * kWave;
        groups = (groups + kWave - 1) / kWave;
    }
    return s;
}

size_t tree_bytes(const TreeShape& s) {
    return static_cast<size_t>(s.offset[s.levels - 1] + s.groups[s.levels - 1] * kWave) *
           sizeof(unsigned long long);
}

}  // namespace

size_t select_workspace_bytes(int64_t m, int64_t r, grass_method method, int replacement) {
    (void)r;
    if (m < 0) m = 0;
    if (method == GRASS_SEL_TOPR) return kHeaderBytes;
    if (replacement) return kHeaderBytes + static_cast<size_t>(m) * 8 + static_cast<size_t>(m) * 4;
    return kHeaderBytes + tree_bytes(tree_shape(m));
}

template <int E, int R>
static grass_status launch_flat(const float* sumsq, int64_t m, int64_t r, grass_method method, int rescale,
                                uint64_t seed, uint64_t refresh_id, int32_t* idx, float* rho,
                                int32_t* status, hipStream_t s) {
    const size_t bytes = static_cast<size_t>((m + kWave * R - 1) / (kWave * R)) * kWave * R * sizeof(unsigned long long);
    if (bytes > 48 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(select_norepl_flat_kernel<E, R>),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(kFlatMaxRows * sizeof(unsigned long long))) != hipSuccess)
        return GRASS_ERR_DEVICE;
    select_norepl_flat_kernel<E, R><<<1, kThreads, bytes, s>>>(sumsq, static_cast<int>(m), static_cast<int>(r),
                                                            method, rescale, seed, refresh_id, idx, rho, status);
    return launch_status();
}

// `status`: the device status word; `body`: select_workspace_bytes(...) - kHeaderBytes bytes of
// device scratch (prefix sums and hit counters, or the tree), 256-byte aligned.
static grass_status launch_select_kernels(const float* sumsq, int64_t m, int64_t r,
                                          grass_method method, int replacement, grass_scale scale,
                                          uint64_t seed, uint64_t refresh_id, int32_t* idx,
                                          float* rho, int32_t* status, char* body, hipStream_t s) {
    if (method == GRASS_SEL_TOPR && m <= kRegMaxRows) {
        const int mi = static_cast<int>(m), ri = static_cast<int>(r);
        if (m <= kThreads) select_topr_reg_kernel<1><<<1, kThreads, 0, s>>>(sumsq, mi, ri, idx, rho, status);
        else if (m <= kRegMaxRows / 4) select_topr_reg_kernel<kRegRows / 4><<<1, kThreads, 0, s>>>(sumsq, mi, ri, idx, rho, status);
        else select_topr_reg_kernel<kRegRows><<<1, kThreads, 0, s>>>(sumsq, mi, ri, idx, rho, status);
        return launch_status();
    }
    if (method == GRASS_SEL_TOPR) {
        select_topr_kernel<<<1, kThreads, 0, s>>>(sumsq, m, r, idx, rho, status);
        return launch_status();
    }
    const int rescale =
        scale == GRASS_SCALE_INV_SQRT_RQ || (scale == GRASS_SCALE_PAPER && replacement);
    if (replacement) {
        unsigned long long* csum = reinterpret_cast<unsigned long long*>(body);
        uint32_t* hits = reinterpret_cast<uint32_t*>(body + static_cast<size_t>(m) * 8);
        if (m <= kRegMaxRows) {
            const size_t bytes = static_cast<size_t>(m) * sizeof(unsigned long long);
            if (m <= kThreads) {
                select_repl_reg_kernel<1><<<1, kThreads, bytes + m * 4, s>>>(
                    sumsq, static_cast<int>(m), r, method, rescale, seed, refresh_id, idx, rho, status, hits);
                return launch_status();
            }
            if (m <= kRegMaxRows / 4) {  // at most 48 KB of LDS
                select_repl_reg_kernel<kRegRows / 4><<<1, kThreads, bytes + m * 4, s>>>(
                    sumsq, static_cast<int>(m), r, method, rescale, seed, refresh_id, idx, rho, status, hits);
                return launch_status();
            }
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(select_repl_reg_kernel<kRegRows>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    static_cast<int>(kRegMaxRows * sizeof(unsigned long long))) != hipSuccess)
                return GRASS_ERR_DEVICE;
            select_repl_reg_kernel<kRegRows><<<1, kThreads, bytes, s>>>(
                sumsq, static_cast<int>(m), r, method, rescale, seed, refresh_id, idx, rho, status, hits);
            return launch_status();
        }
        select_repl_kernel<<<1, kThreads, 0, s>>>(sumsq, m, r, method, rescale, seed, refresh_id,
                                                  idx, rho, status, csum, hits);
        return launch_status();
    }
    if (m > 0 && m <= kFlatMaxRows) {
        return m <= kWave * kWave ? launch_flat<1, 1>(sumsq, m, r, method, rescale, seed, refresh_id, idx, rho, status, s)
               : m <= 2 * kWave * kWave
                   ? launch_flat<1, 2>(sumsq, m, r, method, rescale, seed, refresh_id, idx, rho, status, s)
                   : launch_flat<2, 2>(sumsq, m, r, method, rescale, seed, refresh_id, idx, rho, status, s);
    }
    const TreeShape shape = tree_shape(m);
    const size_t bytes = tree_bytes(shape);
    unsigned long long* ws_tree = reinterpret_cast<unsigned long long*>(body);
    if (bytes <= kLdsTreeBytes) {
        if (bytes > 48 * 1024 &&
            hipFuncSetAttribute(reinterpret_cast<const void*>(select_norepl_kernel<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(bytes)) != hipSuccess)
            return GRASS_ERR_DEVICE;
        select_norepl_kernel<true><<<1, kThreads, bytes, s>>>(
            sumsq, m, r, method, rescale, seed, refresh_id, idx, rho, status, ws_tree, shape);
    } else {
        select_norepl_kernel<false><<<1, kThreads, 0, s>>>(
            sumsq, m, r, method, rescale, seed, refresh_id, idx, rho, status, ws_tree, shape);
    }
    return launch_status();
}

grass_status launch_select(const float* sumsq, int64_t m, int64_t r, grass_method method,
                           int replacement, grass_scale scale, uint64_t seed, uint64_t refresh_id,
                           int32_t* idx, float* rho, void* ws, hipStream_t s) {
    return launch_select_kernels(sumsq, m, r, method, replacement, scale, seed, refresh_id, idx, rho,
                                 static_cast<int32_t*>(ws), static_cast<char*>(ws) + kHeaderBytes, s);
}

size_t select_static_scratch_bytes() { return kStaticScratchBytes; }

// Address of this device's copy of `scratch`, resolved once per device (with that device
// current) and kept; every later call only reads the table.
static grass_status static_scratch_address(char** out) {
    constexpr int kMaxDevices = 64;
    static std::atomic<char*> address[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GRASS_ERR_DEVICE;
    char* p = address[dev].load(std::memory_order_acquire);
    if (!p) {
        void* sym = nullptr;
        if (hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)) != hipSuccess || !sym)
            return GRASS_ERR_DEVICE;
        p = static_cast<char*>(sym);
        address[dev].store(p, std::memory_order_release);  // two first callers store the same value
    }
    *out = p;
    return GRASS_OK;
}

grass_status launch_select_static(const float* sumsq, int64_t m, int64_t r, grass_method method,
                                  int replacement, grass_scale scale, uint64_t seed,
                                  uint64_t refresh_id, int32_t* idx, float* rho, int32_t* status,
                                  hipStream_t s) {
    if (select_workspace_bytes(m, r, method, replacement) > kStaticScratchBytes)
        return GRASS_ERR_WORKSPACE;  // checked by the caller too; never launch past the array
    char* base = nullptr;
    const grass_status st = static_scratch_address(&base);
    if (st != GRASS_OK) return st;
    // Nothing in the scratch has to start at zero: the kernels initialise the prefix sums, the
    // hit counters and every level of the tree (padding included) before they read them, so
    // what the previous call left behind is never seen.
    return launch_select_kernels(sumsq, m, r, method, replacement, scale, seed, refresh_id, idx, rho,
                                 status ? status : reinterpret_cast<int32_t*>(base),
                                 base + kHeaderBytes, s);
}

}  // namespace grass
