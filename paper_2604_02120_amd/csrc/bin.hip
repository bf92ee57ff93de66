// Tile binning on the GPU: duplication with tile|depth keys (paper §2.1(b)), depth sort (§2.1(c))
// and per-tile [start, end) ranges of the sorted list (the per-tile index lists that Alg. 1 and
// Alg. 2 consume).
//
// The result is the list of (tile, Gaussian) pairs ordered by (tile, depth, Gaussian index). It is
// produced without ever sorting 64-bit tile|depth keys:
//   1. the Gaussians themselves are sorted by depth (stable LSD radix sort of N 32-bit keys, so
//      equal depths keep increasing index): this fixes every Gaussian's rank in (depth, index);
//   2. the Gaussians go in rank order to the superblocks of 8 x 8 tiles that they touch, each with a
//      64-bit mask of the tiles, and the masks are then transposed into the tiles' lists ("superblocks"
//      below): no pair is ever sorted.
// Grids of more than 1024 superblocks sort the pairs instead:
//   2. pairs are emitted in rank order, each with its tile id as key (16-bit when the grid has at
//      most 65536 tiles, else 32-bit);
//   3. a stable LSD radix sort of the pairs on the tile id alone (ceil(log2 tiles / 8) passes)
//      then leaves each tile's pairs in rank order, i.e. (depth, index) order.
// Everything is integer work and bit-exact: the covered-tile rectangle is evaluated in
// integer arithmetic (floor((x - r)/16) == (floor(x) - r) >> 4 for integer r).
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
#include <utility>

#include "gsb_internal.h"

namespace gsb {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;                           // per thread
constexpr int kScanTile = kScanThreads * kScanItems;     // 4096 elements per block
constexpr int kScanTopThreads = 1024;
constexpr int kScanTopItems = 4;
constexpr int kScanMaxBlocks = kScanTopThreads * kScanTopItems;   // single-block top level
constexpr int64_t kScanMaxLen = int64_t(kScanTile) * kScanMaxBlocks;  // 16.7M elements
constexpr int kScanSmallBlocks = 1;   // arrays of at most one block: the one-block scan (one launch)

constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;                           // keys per thread (depth sort: or fewer)
constexpr int kSortTile = kSortThreads * kSortItems;     // 4096 keys per block
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;

constexpr int kBigRect = 32;   // mode 0: rectangles with more tiles are emitted by the whole wavefront

// The tile sort's keys are tile ids: 16-bit when the grid has at most 65536 tiles (a 4096 x 4096
// image), which cuts the bytes of the pair emission, the sort passes and the range pass, and
// 32-bit otherwise. The pair order is the same either way.
constexpr int64_t kMaxTiles16 = int64_t(1) << 16;

// Four consecutive keys [idx, idx + 4) with one vector load (idx a multiple of 4; key buffers are
// 256-byte aligned and padded, so a load that straddles the count stays inside the buffer).
__device__ inline uint4 load4(const uint32_t *k, int64_t idx) {
    return *reinterpret_cast<const uint4 *>(k + idx);
}
__device__ inline uint4 load4(const uint16_t *k, int64_t idx) {
    const uint2 v = *reinterpret_cast<const uint2 *>(k + idx);
    return make_uint4(v.x & 0xffffu, v.x >> 16, v.y & 0xffffu, v.y >> 16);
}


struct BinHeader {
    unsigned long long total;     // pairs counted by bin_count
    unsigned long long pairs;     // min(total, capacity), set by bin_fill
    unsigned long long gaussians; // n, for the depth sort
    unsigned long long entries;   // superblock entries
    uint32_t pad[8];
};

// State of one radix sort: the global digit counts of every pass (from the histogram kernel) and
// the ticket counter from which each pass's blocks draw their tile of keys.
constexpr int kMaxPasses = 4;
struct SortState {
    uint32_t hist[kMaxPasses][kRadix];
    uint32_t ticket[kMaxPasses];
    uint32_t pad[64 - kMaxPasses];
};

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

struct Layout {
    // bin_count's part (depends on n only)
    size_t hdr, counts, masks, recs, partials;
    // bin_fill's part
    size_t sorts, dkey_a, dkey_b, dval_a, dval_b, offs, rects, tkey_a, tkey_b, vals_tmp, sortbuf, end;
    size_t sb_mask, sb_idx, sb_counts, sb_groups, sb_table;   // superblock path, in the places of others
};

int64_t sort_blocks(int64_t m, int items = kSortItems) {
    const int64_t tile = int64_t(kSortThreads) * items;
    return (m + tile - 1) / tile;
}

// Superblocks (see below): 8 x 8 tiles, at most kMaxSb of them; entries are taken in chunks.
constexpr int kSbShift = 3, kSbEdge = 1 << kSbShift, kSbTiles = kSbEdge * kSbEdge;
constexpr int kMaxSbBits = 10, kMaxSb = 1 << kMaxSbBits;
// Entries per block: 1024, or 256 where the list is short enough that 1024 would leave most of the
// GPU without a block (the two blocks of 2000 Gaussians took 13 us, the eight take 7).
constexpr int kSbChunkLarge = 1024, kSbChunkSmall = 256;
constexpr int64_t kSbSmallPairs = int64_t(1) << 19;
int sb_chunk_size(int64_t cap) { return cap <= kSbSmallPairs ? kSbChunkSmall : kSbChunkLarge; }
// First entry and first chunk of every superblock, and the ends
constexpr int kSbLists = 8, kSbListRun = 16;
struct SbTable {
    uint32_t start[kMaxSb + 1], chunk[kMaxSb + 1];
    // mode 1: lengths of the lists of the large rectangles' masks, a cache line apart
    alignas(128) unsigned long long listed[kSbLists][16];
};
// chunks that up to `cap` entries can take (a superblock's last chunk may be partial)
int64_t sb_max_chunks(int64_t cap) {
    return cap / sb_chunk_size(cap) + (cap < kMaxSb ? cap : kMaxSb);
}
// Chunks per group: the tiles' pairs before each group of a superblock's chunks are summed once
// (k_tile_scan), so that a chunk adds the counts of its own group's chunks alone.
constexpr int kSbGroup = 64;

// Words of the depth sort's look-back and of the tile sort's histograms, which also hold the counts of
// step 1 of the superblocks
int64_t sort_words(int64_t n, int64_t cap) {
    const int64_t lb_d = int64_t(kMaxPasses) * sort_blocks(n > 0 ? n : 1);
    const int64_t lb_t = sort_blocks(cap > 0 ? cap : 1);
    return kRadix * (lb_d > lb_t ? lb_d : lb_t);
}

Layout layout(int64_t n, int64_t cap) {
    Layout L;
    const size_t nn = size_t(n > 0 ? n : 1), cc = size_t(cap > 0 ? cap : 1);
    size_t o = 0;
    L.hdr = o;       o += align256(sizeof(BinHeader));
    L.counts = o;    o += align256(sizeof(unsigned long long) * nn);
    L.masks = o;     o += align256(sizeof(unsigned long long) * nn);
    L.recs = o;      o += align256(sizeof(uint4) * nn);
    L.partials = o;  o += align256(sizeof(unsigned long long) * kScanMaxBlocks);
    L.sorts = o;     o += align256(sizeof(SortState));
    L.dkey_a = o;    o += align256(sizeof(uint32_t) * nn);
    L.dkey_b = o;    o += align256(sizeof(uint32_t) * nn);
    L.dval_a = o;    o += align256(sizeof(uint32_t) * nn);
    L.dval_b = o;    o += align256(sizeof(uint32_t) * nn);
    L.offs = o;      o += align256(sizeof(unsigned long long) * nn);
    L.rects = o;     o += align256(sizeof(unsigned long long) * nn);
    L.tkey_a = o;    o += align256(sizeof(uint32_t) * cc);
    L.tkey_b = o;    o += align256(sizeof(uint32_t) * cc);
    L.vals_tmp = o;  o += align256(sizeof(uint32_t) * cc);
    // depth sort: look-back words of every pass, [pass][block][digit]; tile sort, afterwards:
    // the per-block digit histograms of one pass, [digit][block]; superblocks, afterwards: the
    // counts [superblock][block] of the entries, then, unless they fit the offsets' place, the
    // tile counts of every chunk, and the groups' sums
    const size_t words = sizeof(uint32_t) * size_t(sort_words(n, cap));
    // (never less than a smaller capacity's: a workspace also serves every shorter list)
    int64_t chunks = sb_max_chunks(int64_t(cc));
    if (int64_t(cc) > kSbSmallPairs && chunks < sb_max_chunks(kSbSmallPairs))
        chunks = sb_max_chunks(kSbSmallPairs);
    const size_t chunk_counts = sizeof(uint16_t) * kSbTiles * size_t(chunks);
    const bool in_offs = chunk_counts <= sizeof(unsigned long long) * nn;
    const size_t before = in_offs ? 0 : align256(chunk_counts);
    const size_t sums = before + sizeof(uint32_t) * kSbTiles * size_t(chunks / kSbGroup + 1);
    L.sortbuf = o;   o += align256(words > sums ? words : sums);
    L.sb_counts = in_offs ? L.offs : L.sortbuf;
    L.sb_groups = L.sortbuf + before;
    // superblock entries: masks in the place of the tile keys, indices in that of the values
    L.sb_mask = L.tkey_a;
    L.sb_idx = L.vals_tmp;
    // the superblock table behind the scans' partial sums (u32 there)
    L.sb_table = L.partials + sizeof(uint32_t) * kScanMaxBlocks;
    L.end = o;
    return L;
}

template <typename T>
T *at(void *ws, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(ws) + off); }

// ------------------------------------------------------------------------------- block scan
// Exclusive scan of one value per thread across the block; `total` receives the block sum.
// `s_wave` holds one slot per wavefront.
template <typename T>
__device__ T block_exclusive_scan(T v, T *s_wave, T &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_wave[w] = x;
    __syncthreads();
    T pre = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        T s = s_wave[i];
        pre += (i < w) ? s : T(0);
        tot += s;
    }
    __syncthreads();
    total = tot;
    return pre + x - v;
}

// ------------------------------------------------------------------------------- device scan
// Exclusive prefix sum, in place. Short arrays: one block walks the array in chunks with a running
// carry. Long arrays: per-block sums, then a per-block scan whose blocks add up the sums before
// them. The total goes to *total_a / *total_b if given. k_scan_top: up to 4096 per-block sums in one
// block.
template <typename T>
__global__ __launch_bounds__(kScanTopThreads) void k_scan_small(T *data, int64_t m,
                                                                unsigned long long *total_a,
                                                                long long *total_b) {
    constexpr int kItems = 16;
    __shared__ T s_wave[kScanTopThreads / 64];
    T carry = 0;
    for (int64_t base = 0; base < m; base += int64_t(kScanTopThreads) * kItems) {
        const int64_t b = base + int64_t(threadIdx.x) * kItems;
        T v[kItems], sum = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            v[k] = (b + k < m) ? data[b + k] : T(0);
            sum += v[k];
        }
        T tot;
        T run = block_exclusive_scan<T>(sum, s_wave, tot) + carry;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            if (b + k < m) data[b + k] = run;
            run += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) {
        if (total_a) *total_a = (unsigned long long)carry;
        if (total_b) *total_b = (long long)carry;
    }
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const T *in, int64_t m, T *partial) {
    __shared__ T s_wave[kScanThreads / 64];
    const int64_t base = int64_t(blockIdx.x) * kScanTile + int64_t(threadIdx.x) * kScanItems;
    T sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < m) sum += in[base + k];
    T tot;
    block_exclusive_scan<T>(sum, s_wave, tot);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

template <typename T>
__global__ __launch_bounds__(kScanTopThreads) void k_scan_top(T *partial, int64_t nb,
                                                               unsigned long long *total_a,
                                                               long long *total_b) {
    __shared__ T s_wave[kScanTopThreads / 64];
    const int64_t base = int64_t(threadIdx.x) * kScanTopItems;
    T v[kScanTopItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kScanTopItems; ++k) {
        v[k] = (base + k < nb) ? partial[base + k] : T(0);
        sum += v[k];
    }
    T tot;
    T run = block_exclusive_scan<T>(sum, s_wave, tot);
#pragma unroll
    for (int k = 0; k < kScanTopItems; ++k) {
        if (base + k < nb) partial[base + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0) {
        if (total_a) *total_a = (unsigned long long)tot;
        if (total_b) *total_b = (long long)tot;
    }
}

// The down pass with the block offsets formed in place: block b sums the per-block totals
// partial[0, b) itself (a few hundred values at most, read from L2) instead of a separate
// single-block scan of them, which saves a launch; the last block writes the total.
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_down_fused(const T *in, T *data, int64_t m,
                                                                   const T *partial, int64_t nb,
                                                                   unsigned long long *total_a,
                                                                   long long *total_b) {
    __shared__ T s_wave[kScanThreads / 64];
    const int64_t blk = blockIdx.x;
    T mine = 0;
    for (int64_t i = threadIdx.x; i < blk; i += kScanThreads) mine += partial[i];
    T offset;
    block_exclusive_scan<T>(mine, s_wave, offset);       // offset = sum of partial[0, blk)
    const int64_t base = blk * kScanTile + int64_t(threadIdx.x) * kScanItems;
    T v[kScanItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < m) ? in[base + k] : T(0);
        sum += v[k];
    }
    T tot;
    T run = block_exclusive_scan<T>(sum, s_wave, tot) + offset;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < m) data[base + k] = run;
        run += v[k];
    }
    if (blk == nb - 1 && threadIdx.x == 0) {
        if (total_a) *total_a = (unsigned long long)(offset + tot);
        if (total_b) *total_b = (long long)(offset + tot);
    }
}

template <typename T>
void launch_scan(T *data, int64_t m, T *partial, unsigned long long *total_a, long long *total_b,
                 hipStream_t s) {
    const int64_t nb = (m + kScanTile - 1) / kScanTile;
    if (nb <= kScanSmallBlocks) {
        k_scan_small<T><<<1, kScanTopThreads, 0, s>>>(data, m, total_a, total_b);
        return;
    }
    k_scan_reduce<T><<<dim3(unsigned(nb)), kScanThreads, 0, s>>>(data, m, partial);
    k_scan_down_fused<T><<<dim3(unsigned(nb)), kScanThreads, 0, s>>>(data, data, m, partial, nb, total_a,
                                                                      total_b);
}

// ------------------------------------------------------------------------------- mode 1
// Binning mode 1 keeps a pair (tile, Gaussian) of the 3-sigma rectangle only when the Gaussian can
// reach alpha >= 1/255 on a pixel of the tile inside the image (opacity-aware extent, a tighter
// binning; images and final T are unchanged because every dropped pair would be skipped):
//   o >= fp32(1/255), and min over the tile's pixel rectangle of Q = d^T Sigma^-1 d <= theta,
//   theta = 2 (e * ln2_up + (m - 1)) + 0.1 with 255 o = m 2^e, m in [1, 2)
// (an upper bound of 2 ln(255 o) without a logarithm, plus a margin far above any exponent error
// of the blend). The minimum of Q over the rectangle of d = (x - px, y - py) is 0 if the rectangle
// contains 0, else it lies on an edge: a 1D quadratic minimised inside the edge or at an end.
// Division-free double-precision tests in a fixed order with contraction off: the decision is
// reproducible bit for bit by any implementation taking the same steps.
constexpr double kLn2Up = 0x1.62e42fefa39fp-1;   // the double just above ln 2
constexpr double kCullMargin = 0.1;

__device__ inline double vis_theta(double o) {
#pragma clang fp contract(off)
    const double z = 255.0 * o;                   // exact: o is an fp32 value
    const unsigned long long bits = (unsigned long long)__double_as_longlong(z);
    const long long e = (long long)((bits >> 52) & 0x7ffull) - 1023;
    const double m = __longlong_as_double(
        (long long)((bits & 0x000fffffffffffffull) | 0x3ff0000000000000ull));
    const double t1 = double(e) * kLn2Up;
    const double t2 = m - 1.0;
    return 2.0 * (t1 + t2) + kCullMargin;
}

// one edge: u fixed at a, v in [c, d]; Q = P a^2 + 2 B a v + R v^2
__device__ inline bool vis_edge(double P, double R, double B, double det, double theta, double a,
                                double c, double d) {
#pragma clang fp contract(off)
    const double ba = B * a;
    const double nba = -ba;
    if (c * R <= nba && nba <= d * R) {           // interior minimum a^2 det / R
        const double lhs = (a * a) * det;
        const double rhs = theta * R;
        return lhs <= rhs;
    }
    const double pa2 = P * (a * a);
    const double qc = (pa2 + (2.0 * ba) * c) + R * (c * c);
    const double qd = (pa2 + (2.0 * ba) * d) + R * (d * d);
    return qc <= theta || qd <= theta;
}

struct GaussVis {
    double x, y, A, B, C, det, theta;
    // Shortcuts that settle most tiles with the same answer as the tests below: with d the point
    // of the tile's rectangle nearest the mean, lmin |d|^2 <= min Q <= Q(d) <= lmax |d|^2 (lmin,
    // lmax the eigenvalues of Sigma^-1). Beyond margins far above the tests' rounding:
    //   |d|^2 > far  => invisible,   |d|^2 < near => visible.
    double far2, near2;
    bool live;                                    // o >= fp32(1/255)
};

__device__ inline GaussVis vis_setup(float2 m, const float *conic, float o) {
#pragma clang fp contract(off)
    GaussVis g;
    g.x = m.x; g.y = m.y;
    g.A = conic[0]; g.B = conic[1]; g.C = conic[2];
    g.live = o >= 1.0f / 255.0f;
    g.det = g.A * g.C - g.B * g.B;
    g.theta = vis_theta(double(o));
    g.far2 = INFINITY;                            // no shortcut unless positive definite
    g.near2 = -1.0;
    if (g.A > 0.0 && g.det > 0.0) {
        const double h = 0.5 * (g.A + g.C), r = sqrt(0.25 * (g.A - g.C) * (g.A - g.C) + g.B * g.B);
        const double lmax = (h + r) * (1.0 + 1e-9);
        const double lmin = (g.det / (h + r)) * (1.0 - 1e-9);
        g.far2 = (g.theta + 1e-6 * (1.0 + g.theta)) / lmin;
        g.near2 = (g.theta - 1e-6 * (1.0 + g.theta)) / lmax;
    }
    return g;
}

__device__ inline bool tile_visible(const GaussVis &g, int32_t tx, int32_t ty, int32_t W,
                                    int32_t H) {
#pragma clang fp contract(off)
    if (!g.live) return false;
    const int32_t px1 = tx * kTile + kTile - 1 < W - 1 ? tx * kTile + kTile - 1 : W - 1;
    const int32_t py1 = ty * kTile + kTile - 1 < H - 1 ? ty * kTile + kTile - 1 : H - 1;
    const double dxl = g.x - double(px1), dxh = g.x - double(tx * kTile);
    const double dyl = g.y - double(py1), dyh = g.y - double(ty * kTile);
    if (dxl <= 0.0 && 0.0 <= dxh && dyl <= 0.0 && 0.0 <= dyh) return true;
    const double cx = dxl > 0.0 ? dxl : (dxh < 0.0 ? dxh : 0.0);
    const double cy = dyl > 0.0 ? dyl : (dyh < 0.0 ? dyh : 0.0);
    const double d2 = cx * cx + cy * cy;
    if (d2 > g.far2) return false;
    if (d2 < g.near2) return true;
    // only the edges facing the mean can hold the minimum (at most one in x, one in y)
    if (dxl > 0.0 && vis_edge(g.A, g.C, g.B, g.det, g.theta, dxl, dyl, dyh)) return true;
    if (dxh < 0.0 && vis_edge(g.A, g.C, g.B, g.det, g.theta, dxh, dyl, dyh)) return true;
    if (dyl > 0.0 && vis_edge(g.C, g.A, g.B, g.det, g.theta, dyl, dxl, dxh)) return true;
    if (dyh < 0.0 && vis_edge(g.C, g.A, g.B, g.det, g.theta, dyh, dxl, dxh)) return true;
    return false;
}

// The same decision in FP32 where it is clear. The smallest Q over the tile's rectangle is at one of
// two points (the nearest dx with its best dy, the nearest dy with its best dx; 0 if the mean lies
// inside); evaluated in FP32 its error is below 2^-16 of its (positive) terms, theta's below 2^-18 of
// it. Between the two bounds, and for a conic that is not definite, the tests above decide. (They
// take about 90 double-precision operations a tile: 291 us of 3 M Gaussians at 4K, now 190.)
struct Vis32 {
    float x, y, A, B, C, o, rA, rC;
    float lo, hi;                                 // theta less and plus its error; -inf, inf: unclear
};
__device__ inline Vis32 vis32_setup(float2 m, const float *conic, float o, Rect *cand, const Rect &R) {
    Vis32 g;
    g.x = m.x; g.y = m.y;
    g.A = conic[0]; g.B = conic[1]; g.C = conic[2];
    g.o = o;
    const float theta = float(vis_theta(double(o)));
    const float bb = g.B * g.B;
    const float det = fmaf(g.A, g.C, -bb) - fmaf(g.B, g.B, -bb);
    // (in a range where none of the products below overflows and a pixel is a pixel)
    const bool definite = g.A > 1e-18f && g.A < 1e18f && g.C > 1e-18f && g.C < 1e18f && det > 0.f &&
                          fabsf(g.x) < 0x1p20f && fabsf(g.y) < 0x1p20f;
    g.rA = __builtin_amdgcn_rcpf(g.A);
    g.rC = __builtin_amdgcn_rcpf(g.C);
    g.lo = definite ? theta * (1.0f - 0x1p-18f) : -INFINITY;
    g.hi = definite ? theta * (1.0f + 0x1p-18f) : INFINITY;
    if (cand) {
        // candidates: the rectangle cut to the bounding box of {Q <= theta}, with room for rounding
        *cand = R;
        if (!(o >= 1.0f / 255.0f)) {
            *cand = Rect{0, 0, 0, 0};
        } else if (definite) {
            const float hx = fminf(sqrtf(theta * g.C / det) * 1.001f + 1.5f, 1e8f);
            const float hy = fminf(sqrtf(theta * g.A / det) * 1.001f + 1.5f, 1e8f);
            const auto lo = [](float v) { return int64_t(floorf((v - 15.0f) * 0.0625f)); };
            const auto hi = [](float v) { return int64_t(floorf(v * 0.0625f)) + 1; };
            cand->tx0 = int32_t(clampi(lo(g.x - hx), R.tx0, R.tx1));
            cand->tx1 = int32_t(clampi(hi(g.x + hx), cand->tx0, R.tx1));
            cand->ty0 = int32_t(clampi(lo(g.y - hy), R.ty0, R.ty1));
            cand->ty1 = int32_t(clampi(hi(g.y + hy), cand->ty0, R.ty1));
        }
    }
    return g;
}
__device__ inline bool tile_visible(const Vis32 &g, int32_t tx, int32_t ty, int32_t W, int32_t H) {
    const int32_t px1 = tx * kTile + kTile - 1 < W - 1 ? tx * kTile + kTile - 1 : W - 1;
    const int32_t py1 = ty * kTile + kTile - 1 < H - 1 ? ty * kTile + kTile - 1 : H - 1;
    const float dxl = g.x - float(px1), dxh = g.x - float(tx * kTile);
    const float dyl = g.y - float(py1), dyh = g.y - float(ty * kTile);
    const float a = fminf(fmaxf(0.0f, dxl), dxh), b = fminf(fmaxf(0.0f, dyl), dyh);
    const float ba = g.B * a, bb = g.B * b;
    const float v = fminf(fmaxf(-ba * g.rC, dyl), dyh), u = fminf(fmaxf(-bb * g.rA, dxl), dxh);
    const float s1 = fmaf(g.A * a, a, g.C * v * v), s2 = fmaf(g.C * b, b, g.A * u * u);
    const float q1 = fmaf(2.0f * ba, v, s1), q2 = fmaf(2.0f * bb, u, s2);
    const bool in = fmaf(s1, 0x1p-16f, q1) < g.lo || fmaf(s2, 0x1p-16f, q2) < g.lo;
    const bool out = fmaf(s1, -0x1p-16f, q1) > g.hi && fmaf(s2, -0x1p-16f, q2) > g.hi;
    if (in || out) return in;
    const float conic[3] = {g.A, g.B, g.C};
    return tile_visible(vis_setup(make_float2(g.x, g.y), conic, g.o), tx, ty, W, H);
}

// visible-tile masks: a Gaussian with at most this many candidates keeps its answer as one bit per
// candidate (row-major), so that emission needs no second test
constexpr uint32_t kMaskBits = 64;

// The same mask where superblocks follow: a byte per row, of rectangles of up to 8 x 8 tiles (what a
// superblock needs of it is then two shifts away; from the other form it took a loop over the rows,
// in each of the two kernels that ask: 73 and 117 us, now 45 and 99)
__device__ inline bool sb_big(const Rect &R) { return R.tx1 - R.tx0 > 8 || R.ty1 - R.ty0 > 8; }
__device__ inline unsigned long long sb_form(const Rect &R, unsigned long long mask) {
    const int w = R.tx1 - R.tx0, h = R.ty1 - R.ty0;
    const uint32_t row = (1u << w) - 1u;
    uint32_t half[2] = {0u, 0u};
#pragma unroll
    for (int y = 0; y < 8; ++y) {
        if (y < h) half[y >> 2] |= (uint32_t(mask) & row) << (8 * (y & 3));
        mask >>= w;
    }
    return (static_cast<unsigned long long>(half[1]) << 32) | half[0];
}

// ------------------------------------------------------------------------------- balanced pairs
// The candidate tiles of a wavefront's 64 rectangles are enumerated in chunks of 64, one candidate
// per lane, whatever the rectangles' sizes: a candidate's rectangle (its owner lane) is found by a
// binary search over the wavefront's exclusive prefix of areas, and the tile from the index within
// that rectangle (row-major). Owners' visibility parameters sit in LDS.
struct WaveCands {
    uint32_t excl;     // this lane's exclusive prefix of areas
    uint32_t total;    // the wavefront's number of candidates
};

__device__ inline WaveCands wave_cands(uint32_t area) {
    const int lane = threadIdx.x & 63;
    uint32_t x = area;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return WaveCands{x - area, uint32_t(__shfl(x, 63, 64))};
}

// the lane owning candidate k: the last lane whose exclusive prefix is <= k
__device__ inline int cand_owner(uint32_t excl, uint32_t k) {
    int o = 0;
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1)
        if (uint32_t(__shfl(int(excl), o + step, 64)) <= k) o += step;
    return o;
}

// a / b and a % b for a < 2^25, 0 < b < 2^13: a float quotient (error < 8) corrected exactly
__device__ inline void divmod_small(uint32_t a, uint32_t b, uint32_t &q, uint32_t &r) {
    uint32_t qq = uint32_t(float(a) * __builtin_amdgcn_rcpf(float(b)));
    int32_t rr = int32_t(a) - int32_t(qq * b);
    while (rr < 0) { --qq; rr += int32_t(b); }
    while (rr >= int32_t(b)) { ++qq; rr -= int32_t(b); }
    q = qq;
    r = uint32_t(rr);
}

// lanes [s, e) of a 64-bit lane mask (0 <= s <= e <= 64)
__device__ inline unsigned long long lane_range(int s, int e) {
    const unsigned long long hi = e >= 64 ? ~0ull : ((1ull << e) - 1ull);
    const unsigned long long lo = s >= 64 ? ~0ull : ((1ull << s) - 1ull);
    return hi & ~lo;
}

// candidates of owner lane l that fall in the chunk [cb, cb + 64)
__device__ inline unsigned long long owner_run(uint32_t excl, uint32_t area, uint32_t cb) {
    const int64_t s0 = int64_t(excl) - int64_t(cb), e0 = s0 + int64_t(area);
    const int s = int(s0 < 0 ? 0 : (s0 > 64 ? 64 : s0)), e = int(e0 < 0 ? 0 : (e0 > 64 ? 64 : e0));
    return lane_range(s, e);
}

// Pair counts per Gaussian. Mode 0: the rectangle's area. Mode 1: its visible candidates, with
// the candidates of each wavefront balanced over its lanes; a Gaussian with at most kMaskBits
// candidates also records which ones are visible (masks).
// A Gaussian's pair count and emission rectangle in one 16-byte record, stored by Gaussian index:
// the depth sort's last pass gathers both with one load and lays them out in rank order, so that
// the pair emission reads them in order instead of gathering means and radii by rank. Tile
// coordinates are at most 4096 and fit 16 bits.
__device__ inline uint4 count_rect(unsigned long long cnt, const Rect &R) {
    return make_uint4(uint32_t(cnt), uint32_t(cnt >> 32), uint32_t(R.tx0) | (uint32_t(R.tx1) << 16),
                      uint32_t(R.ty0) | (uint32_t(R.ty1) << 16));
}
__device__ inline Rect unpack_rect(unsigned long long p) {
    const uint32_t x = uint32_t(p), y = uint32_t(p >> 32);
    return Rect{int32_t(x & 0xffffu), int32_t(x >> 16), int32_t(y & 0xffffu), int32_t(y >> 16)};
}

// Mode 1, the Gaussian i of this thread (i >= n: none; every lane of a wavefront takes part).
__device__ inline unsigned long long count_visible(const float2 *means, const int32_t *radii,
                                                   const float *conics, const float *opac, int64_t i,
                                                   int64_t n, int32_t gx, int32_t gy, int32_t W,
                                                   int32_t H, Vis32 *s_vis,
                                                   unsigned long long *counts,
                                                   unsigned long long *masks, uint4 *recs) {
    const bool valid = i < n;
    Rect CR{0, 0, 0, 0};
    Vis32 g{};
    if (valid) {
        const float2 m = means[i];
        g = vis32_setup(m, conics + 3 * i, opac[i], &CR, tile_rect(m.x, m.y, radii[i], gx, gy));
    }
    s_vis[threadIdx.x] = g;   // read only by this wavefront's lanes
    __builtin_amdgcn_wave_barrier();
    const int w = CR.tx1 - CR.tx0;
    const uint32_t area = uint32_t(w * (CR.ty1 - CR.ty0));
    const WaveCands wc = wave_cands(area);
    const int lane = threadIdx.x & 63, wbase = threadIdx.x & ~63;
    unsigned long long cnt = 0, mask = 0;
    for (uint32_t cb = 0; cb < wc.total; cb += 64) {
        const uint32_t k = cb + lane;
        const bool act = k < wc.total;
        const int o = cand_owner(wc.excl, act ? k : wc.total - 1);
        const uint32_t jl = (act ? k : 0u) - uint32_t(__shfl(int(wc.excl), o, 64));
        const int ow = __shfl(w, o, 64), otx0 = __shfl(CR.tx0, o, 64), oty0 = __shfl(CR.ty0, o, 64);
        uint32_t qy = 0, rx = 0;
        if (act) divmod_small(jl, uint32_t(ow), qy, rx);
        bool v = false;
        if (act) v = tile_visible(s_vis[wbase + o], otx0 + int(rx), oty0 + int(qy), W, H);
        // as an owner: my candidates in this chunk are lanes [rs, re)
        const unsigned long long mine = __ballot(v) & owner_run(wc.excl, area, cb);
        cnt += __popcll(mine);
        if (area <= kMaskBits && mine) {
            const int64_t rs = int64_t(wc.excl) - int64_t(cb);
            const int s0 = rs > 0 ? int(rs) : 0;
            const int j0 = rs > 0 ? 0 : int(-rs);      // my first candidate index in this chunk
            mask |= (mine >> s0) << j0;
        }
    }
    if (valid) {
        if (counts) {
            counts[i] = cnt;
            masks[i] = mask;
        }
        // superblocks: the mask (0 where it has no room for the rectangle) in the count's place
        recs[i] = count_rect(counts ? cnt : sb_big(CR) ? 0ull : sb_form(CR, mask), CR);
    }
    return cnt;
}

// A block counts the pairs of `iters` x kThreads Gaussians and leaves their sum in partial[block] (a
// single block writes the total itself), so that no other pass reads the counts; they are stored
// only where the pair sort needs them (counts not null).
template <int kMode, int kThreads>
__global__ __launch_bounds__(kThreads) void k_bin_count(const float2 *means, const int32_t *radii,
                                                        const float *conics, const float *opac,
                                                        int64_t n, int iters, int32_t gx,
                                                        int32_t gy, int32_t W, int32_t H,
                                                        unsigned long long *counts,
                                                        unsigned long long *masks, uint4 *recs,
                                                        unsigned long long *partial,
                                                        unsigned long long *total_a,
                                                        long long *total_b) {
    __shared__ Vis32 s_vis[kMode == 1 ? kThreads : 1];
    __shared__ unsigned long long s_wave[kThreads / 64];
    const int64_t i0 = int64_t(blockIdx.x) * iters * kThreads + threadIdx.x;
    unsigned long long sum = 0, all;
    if constexpr (kMode == 0) {
#pragma unroll 4
        for (int it = 0; it < iters; ++it) {
            const int64_t i = i0 + int64_t(it) * kThreads;
            if (i >= n) continue;
            const float2 m = means[i];
            const Rect R = tile_rect(m.x, m.y, radii[i], gx, gy);
            const unsigned long long cnt =
                (unsigned long long)(R.tx1 - R.tx0) * (unsigned long long)(R.ty1 - R.ty0);
            if (counts) counts[i] = cnt;
            recs[i] = count_rect(cnt, R);
            sum += cnt;
        }
    } else {
        for (int it = 0; it < iters; ++it) {
            const int64_t i = i0 + int64_t(it) * kThreads;
            if (i - threadIdx.x >= n) break;                 // block-uniform
            sum += count_visible(means, radii, conics, opac, i, n, gx, gy, W, H, s_vis, counts,
                                 masks, recs);
        }
    }
    block_exclusive_scan<unsigned long long>(sum, s_wave, all);
    if (threadIdx.x == 0) {
        if (gridDim.x > 1) {
            partial[blockIdx.x] = all;
        } else {
            *total_a = all;
            *total_b = (long long)all;
        }
    }
}

// Depth keys: the float's bits, made order-preserving for any sign (a no-op flip of the sign bit
// for the positive depths of the contract).
__device__ inline uint32_t depth_key(float d) {
    const uint32_t b = __float_as_uint(d);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Emits the pairs of the Gaussian of rank j at offs[j]: tile id as key, Gaussian index as value.
// The block's 256 consecutive ranks own one contiguous output segment; when it fits in LDS the
// pairs are assembled there and written out in order (coalesced), otherwise straight to memory.
// A lane emits its own rectangle when it is small; larger ones are emitted by the whole wavefront
// together, one after the other.
// Pairs staged per block: 4096, or 6144 where a block's 256 ranks are expected to emit more than
// 7/8 of 4096 (the host estimates it from the capacity per Gaussian). Blocks whose segment does
// not fit write straight to memory, uncoalesced: at 4K 82% of the blocks overflow 4096 (binning
// 1.211 -> 1.151 ms with 6144), while at 1080p the larger stage only costs occupancy.
constexpr int kFillStage = 4096, kFillStageLarge = 6144;

template <typename K, int kStage> struct PairSink {
    K *keys;                         // global
    uint32_t *vals;
    K *skey;                         // LDS segment, or null
    uint32_t *sval;
    unsigned long long seg0, cap;    // first output index of the block, capacity
    __device__ inline void put(unsigned long long o, uint32_t key, uint32_t val) const {
        if (skey) {
            if (o - seg0 >= (unsigned long long)kStage) return;   // never for consistent counts
            skey[o - seg0] = K(key);
            sval[o - seg0] = val;
        } else if (o < cap) {
            keys[o] = K(key);
            vals[o] = val;
        }
    }
};

template <typename K, int kStage>
__global__ __launch_bounds__(256) void k_bin_fill(const float2 *means, const float *conics,
                                                  const float *opac,
                                                  int32_t mode, int32_t W, int32_t H,
                                                  const uint32_t *sorted_idx, int64_t n,
                                                  int32_t gx, int32_t gy,
                                                  const unsigned long long *offs,
                                                  const unsigned long long *counts,
                                                  const unsigned long long *masks,
                                                  const unsigned long long *rank_rects,
                                                  BinHeader *hdr, int64_t cap, K *keys,
                                                  uint32_t *vals, int32_t *status) {
    __shared__ K s_key[kStage];
    __shared__ uint32_t s_val[kStage];
    const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j == 0) {
        const unsigned long long total = hdr->total;
        hdr->pairs = total < (unsigned long long)cap ? total : (unsigned long long)cap;
        if (total > (unsigned long long)cap) *status = GSB_ERR_CAPACITY;
    }
    const int64_t j0 = int64_t(blockIdx.x) * blockDim.x;
    if (j0 >= n) return;   // block-uniform (only the single block of an empty launch)
    const bool valid = j < n;
    const uint32_t i = valid ? sorted_idx[j] : 0u;
    // the rectangle to emit from (laid out in rank order by the depth sort): mode 0 the 3-sigma
    // one, mode 1 the candidates (vis32_setup)
    Rect R{0, 0, 0, 0};
    GaussVis g{};
    unsigned long long base = 0, vmask = 0;
    if (valid) {
        R = unpack_rect(rank_rects[j]);
        base = offs[j];
        if (mode != 0) {
            g = vis_setup(means[i], conics + 3 * int64_t(i), opac[i]);
            vmask = masks[i];
        }
    }
    // the block's segment: [first rank's offset, last rank's offset + its count)
    const int64_t jl = (j0 + int64_t(blockDim.x) < n ? j0 + int64_t(blockDim.x) : n) - 1;
    const unsigned long long seg0 = offs[j0];
    const unsigned long long seg1 = offs[jl] + counts[sorted_idx[jl]];
    const unsigned long long ucap = (unsigned long long)cap;
    const bool staged = (seg1 - seg0) <= (unsigned long long)kStage && seg1 <= ucap;
    const PairSink<K, kStage> sink{keys, vals, staged ? s_key : nullptr, staged ? s_val : nullptr,
                                   seg0, ucap};

    const int w = R.tx1 - R.tx0;
    const int area = w * (R.ty1 - R.ty0);
    // small rectangles: the lane emits its own (mode 1: the recorded visible candidates); large
    // ones: the whole wavefront together, one after the other (mode 1: testing each candidate)
    const bool big = mode == 0 ? area > kBigRect : area > int(kMaskBits);
    if (!big) {
        unsigned long long o = base;
        if (mode == 0) {
            for (int32_t ty = R.ty0; ty < R.ty1; ++ty)
                for (int32_t tx = R.tx0; tx < R.tx1; ++tx, ++o)
                    sink.put(o, uint32_t(int64_t(ty) * gx + tx), i);
        } else {
            // row by row: bits [r w, r w + w) of the mask are row r of the candidates
            const unsigned long long rowm = w >= 64 ? ~0ull : ((1ull << w) - 1ull);
            for (int32_t ty = R.ty0, sh = 0; ty < R.ty1; ++ty, sh += w) {
                for (unsigned long long mk = (vmask >> sh) & rowm; mk; mk &= mk - 1, ++o) {
                    const int bx = __ffsll((long long)mk) - 1;
                    sink.put(o, uint32_t(int64_t(ty) * gx + (R.tx0 + bx)), i);
                }
            }
        }
    }
    unsigned long long todo = __ballot(big);
    const int lane = threadIdx.x & 63;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    while (todo) {
        const int src = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        const int stx0 = __builtin_amdgcn_readlane(R.tx0, src);
        const int sty0 = __builtin_amdgcn_readlane(R.ty0, src);
        const int sw = __builtin_amdgcn_readlane(w, src);
        const int sarea = __builtin_amdgcn_readlane(area, src);
        const uint32_t si = __builtin_amdgcn_readlane(i, src);
        const unsigned long long sbase =
            ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane(uint32_t(base >> 32), src) << 32) |
            (uint32_t)__builtin_amdgcn_readlane(uint32_t(base), src);
        if (mode == 0) {
            for (int k = lane; k < sarea; k += 64) {
                const int ty = sty0 + k / sw, tx = stx0 + k % sw;
                sink.put(sbase + k, uint32_t(int64_t(ty) * gx + tx), si);
            }
        } else {
            GaussVis sg;
            sg.x = __shfl(g.x, src); sg.y = __shfl(g.y, src);
            sg.A = __shfl(g.A, src); sg.B = __shfl(g.B, src); sg.C = __shfl(g.C, src);
            sg.det = __shfl(g.det, src); sg.theta = __shfl(g.theta, src);
            sg.far2 = __shfl(g.far2, src); sg.near2 = __shfl(g.near2, src);
            sg.live = true;
            unsigned long long o = sbase;       // visible candidates in row-major order
            for (int k0 = 0; k0 < sarea; k0 += 64) {
                const int k = k0 + lane;
                const int ty = sty0 + k / sw, tx = stx0 + k % sw;
                const bool v = k < sarea && tile_visible(sg, tx, ty, W, H);
                const unsigned long long vb = __ballot(v);
                if (v) sink.put(o + __popcll(vb & lt_mask), uint32_t(int64_t(ty) * gx + tx), si);
                o += __popcll(vb);
            }
        }
    }
    if (staged) {   // block-uniform
        __syncthreads();
        const int len = int(seg1 - seg0);
        for (int k = threadIdx.x; k < len; k += blockDim.x) {
            keys[seg0 + k] = s_key[k];
            vals[seg0 + k] = s_val[k];
        }
    }
}

// ------------------------------------------------------------------------------- radix sort
// Stable LSD radix sort of (key, u32 value) on 8-bit digits. The depth sort (u32 keys) takes one
// kernel per pass plus one histogram kernel per sort (a "onesweep" organisation with decoupled
// look-back):
//   * k_sort_hist reads the keys once and accumulates the global digit counts of every pass (at
//     most 256 blocks, so few blocks add into each global count); it also clears the look-back
//     words of every pass.
//   * k_radix_pass<chained>, one launch per pass: each block draws the index of its tile of 4096 keys from
//     a ticket counter (so a block only ever waits on tiles whose blocks are already running),
//     ranks its keys stably in LDS, publishes its per-digit counts, and walks back over the
//     preceding tiles' published words (16 per step) until it meets an inclusive prefix. A digit's global
//     start is the exclusive scan of the pass's digit counts plus that prefix. Keys are then
//     written out in digit order (contiguous runs, so the global writes coalesce).
// The tile sort (u16 or u32 keys, see sort_tiles) runs each pass as a per-block histogram, its
// scan and k_radix_pass<unchained>, which reads its digit offsets instead of looking back.
// A look-back word is flag << 30 | value: flag 1 = the tile's own count, 2 = inclusive prefix.
// Every wait is bounded; an expired wait reports GSB_ERR_INTERNAL in the status word instead of
// hanging. The element count is read from device memory (*count).
constexpr uint32_t kFlagAgg = 1u << 30, kFlagInc = 2u << 30, kValMask = (1u << 30) - 1u;
constexpr uint32_t kSpinLimit = 1u << 22;
constexpr int kLookback = 16;           // preceding tiles read per look-back step
constexpr int kHistBlocks = 256;        // histogram kernel: at most this many blocks

// The keys are made here from the depths (and written with the identity values).
template <int kItems>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const float *depths, uint32_t *keys_io,
                                                            uint32_t *vals_out,
                                                            const unsigned long long *count,
                                                            int passes, SortState *st,
                                                            uint32_t *lookback, int64_t nblk) {
    __shared__ uint32_t s_h[kMaxPasses][kRadix];
    const int t = threadIdx.x;
    for (int p = 0; p < passes; ++p) s_h[p][t] = 0u;
    // this block's tiles: blockIdx.x, + gridDim.x, ... (their look-back words are cleared here)
    for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x)
        for (int p = 0; p < passes; ++p) lookback[(int64_t(p) * nblk + b) * kRadix + t] = 0u;
    __syncthreads();
    const int64_t P = int64_t(*count);
    for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int64_t base = b * (kSortThreads * kItems);
        if (base >= P) break;
        // four consecutive entries per thread and step: the keys and identity values are stored
        // with 16-byte writes (the workspace buffers are 256-byte aligned)
#pragma unroll
        for (int k = 0; k < kItems / 4; ++k) {
            const int64_t idx = base + 4 * (int64_t(k) * kSortThreads + t);
            if (idx >= P) continue;
            uint32_t key[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) key[j] = idx + j < P ? depth_key(depths[idx + j]) : 0u;
            if (idx + 4 <= P) {
                *reinterpret_cast<uint4 *>(keys_io + idx) = make_uint4(key[0], key[1], key[2], key[3]);
                const uint32_t i0 = uint32_t(idx);
                *reinterpret_cast<uint4 *>(vals_out + idx) = make_uint4(i0, i0 + 1, i0 + 2, i0 + 3);
            } else {
                for (int j = 0; idx + j < P; ++j) {
                    keys_io[idx + j] = key[j];
                    vals_out[idx + j] = uint32_t(idx + j);
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (idx + j >= P) break;
                for (int p = 0; p < passes; ++p)
                    atomicAdd(&s_h[p][(key[j] >> (kRadixBits * p)) & (kRadix - 1)], 1u);
            }
        }
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p)
        if (s_h[p][t]) atomicAdd(&st->hist[p][t], s_h[p][t]);
}

// Per-block digit histogram of one pass, stored digit-major ([digit][block]) so that one
// exclusive scan yields every block's output offset per digit.
template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_block_hist(const K *keys,
                                                             const unsigned long long *count,
                                                             int shift, uint32_t *hist,
                                                             int64_t nblk) {
    __shared__ uint32_t s_h[kRadix];
    const int t = threadIdx.x;
    s_h[t] = 0;
    __syncthreads();
    const int64_t P = int64_t(*count);
    const int64_t base = int64_t(blockIdx.x) * kSortTile;
    // four keys per load (order does not matter to a histogram), all loads issued before any is
    // counted (from index 0 where past P: entries >= P are ignored)
    uint4 q[kSortItems / 4];
#pragma unroll
    for (int k = 0; k < kSortItems / 4; ++k) {
        const int64_t idx = base + 4 * (int64_t(k) * kSortThreads + t);
        q[k] = load4(keys, idx < P ? idx : 0);
    }
#pragma unroll
    for (int k = 0; k < kSortItems / 4; ++k) {
        const int64_t idx = base + 4 * (int64_t(k) * kSortThreads + t);
        if (idx < P) {
            const uint4 v = q[k];
            atomicAdd(&s_h[(v.x >> shift) & (kRadix - 1)], 1u);
            if (idx + 1 < P) atomicAdd(&s_h[(v.y >> shift) & (kRadix - 1)], 1u);
            if (idx + 2 < P) atomicAdd(&s_h[(v.z >> shift) & (kRadix - 1)], 1u);
            if (idx + 3 < P) atomicAdd(&s_h[(v.w >> shift) & (kRadix - 1)], 1u);
        }
    }
    __syncthreads();
    hist[int64_t(t) * nblk + blockIdx.x] = s_h[t];
}

__device__ inline void lb_publish(uint32_t *w, uint32_t v) {
    __hip_atomic_store(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint32_t lb_read(const uint32_t *w) {
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// kRankCounts (last pass of the depth sort): also writes, at each Gaussian's rank, the number of
// pairs it emits (unless rank_counts is null) and its emission rectangle (from the record
// recs_by_idx[value]) into rank_counts and rank_rects.
// kChained: the block's tile comes from `ticket` and its digit offsets from the look-back over
// `lookback` plus the pass's digit counts `ghist`; otherwise tile = blockIdx.x and the offsets are
// read from `hist_off` ([digit][block], the exclusive scan of the per-block histograms).
template <bool kChained, bool kRankCounts, typename K = uint32_t, int kItems = kSortItems>
__global__ __launch_bounds__(kSortThreads) void k_radix_pass(
    const K *kin, const uint32_t *vin, K *kout, uint32_t *vout,
    const unsigned long long *count, int shift, const uint32_t *ghist, uint32_t *lookback,
    uint32_t *ticket, int32_t *status, const uint32_t *hist_off, int64_t nblk,
    const uint4 *recs_by_idx, unsigned long long *rank_counts, unsigned long long *rank_rects) {
    constexpr int kTileKeys = kSortThreads * kItems;
    __shared__ uint32_t s_wcnt[kSortThreads / 64][kRadix];  // per-wave digit counts, then prefixes
    __shared__ uint32_t s_dstart[kRadix];                     // block-local start of each digit
    __shared__ uint32_t s_gofs[kRadix];                       // global start of each digit
    __shared__ uint32_t s_wave[kSortThreads / 64];
    __shared__ K s_key[kTileKeys];
    __shared__ uint32_t s_val[kTileKeys];
    __shared__ uint32_t s_tile;

    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (kChained && t == 0) s_tile = atomicAdd(ticket, 1u);
#pragma unroll
    for (int d = 0; d < kSortThreads / 64; ++d) s_wcnt[d][t] = 0;
    __syncthreads();
    const int64_t tile = kChained ? int64_t(s_tile) : int64_t(blockIdx.x);
    const int64_t P = int64_t(*count);
    const int64_t base = tile * kTileKeys;
    if (base >= P) return;   // block-uniform; every later ticket is empty too

    // Wave w ranks keys [base + 1024 w, base + 1024 (w + 1)) in 16 steps of 64 consecutive keys,
    // so rank order within the wave is index order. All loads are issued first, from an index
    // clamped into [base, P) (validity applied afterwards), so that they are in flight together.
    uint32_t key[kItems], val[kItems], loc[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t idx = base + int64_t(w) * (kItems * 64) + k * 64 + lane;
        const int64_t ci = idx < P ? idx : P - 1;   // P > base here
        key[k] = uint32_t(kin[ci]);
        val[k] = vin[ci];
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t idx = base + int64_t(w) * (kItems * 64) + k * 64 + lane;
        const bool valid = idx < P;
        const uint32_t d = (key[k] >> shift) & (kRadix - 1);
        // lanes holding the same digit: intersect, over the digit's bits, the lanes whose bit
        // equals this lane's (the ballot of the set bits, flipped where this lane's bit is clear),
        // on the two 32-bit halves of the mask (written in place: from a function of its own the
        // compiler makes two more instructions per bit)
        const unsigned long long vmask = __builtin_amdgcn_ballot_w64(valid);
        uint32_t plo = uint32_t(vmask), phi = uint32_t(vmask >> 32);
        const uint32_t nd = ~d;
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            const uint32_t flip = uint32_t(int32_t(nd << (31 - b)) >> 31);  // ones if bit b clear
            const unsigned long long vote = __builtin_amdgcn_ballot_w64(flip == 0u);
            plo &= uint32_t(vote) ^ flip;
            phi &= uint32_t(vote >> 32) ^ flip;
        }
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
        uint32_t prior = 0;
        if (valid) prior = s_wcnt[w][d];
        if (valid && rank == 0) s_wcnt[w][d] = prior + uint32_t(__popc(plo) + __popc(phi));
        loc[k] = prior + rank;
    }
    __syncthreads();
    // thread t = digit t: exclusive prefix over waves, then the tile's count of digit t
    uint32_t c[kSortThreads / 64], run = 0;
#pragma unroll
    for (int i = 0; i < kSortThreads / 64; ++i) {
        c[i] = s_wcnt[i][t];
        s_wcnt[i][t] = run;
        run += c[i];
    }
    uint32_t excl = 0;
    uint32_t *my = kChained ? lookback + tile * kRadix + t : nullptr;
    if (kChained) lb_publish(my, (tile == 0 ? kFlagInc : kFlagAgg) | run);
    if (kChained && tile > 0) {
        // walk back over the preceding tiles kLookback at a time (independent loads), summing
        // their counts up to the first inclusive prefix; a tile that has published nothing yet is
        // waited for
        int64_t j = tile - 1;
        uint32_t spins = 0;
        bool done = false;
        while (!done) {
            uint32_t wv[kLookback];
#pragma unroll
            for (int k = 0; k < kLookback; ++k)
                wv[k] = (j - k >= 0) ? lb_read(lookback + (j - k) * kRadix + t) : kFlagInc;
            int k = 0;
            for (; k < kLookback; ++k) {
                const uint32_t flag = wv[k] & ~kValMask;
                if (flag == 0u) break;              // not published yet: re-read from here
                excl += wv[k] & kValMask;
                if (flag == kFlagInc) { done = true; break; }
            }
            if (done) break;
            j -= k;
            if (k < kLookback) {
                if (++spins > kSpinLimit) {         // never expected: report instead of hanging
                    *status = GSB_ERR_INTERNAL;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        lb_publish(my, kFlagInc | (excl + run));
    }
    uint32_t tot;
    if constexpr (kChained) {
        const uint32_t dglob = block_exclusive_scan<uint32_t>(ghist[t], s_wave, tot);
        s_gofs[t] = dglob + excl;
    } else {
        s_gofs[t] = hist_off[int64_t(t) * nblk + tile];
    }
    s_dstart[t] = block_exclusive_scan<uint32_t>(run, s_wave, tot);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t idx = base + int64_t(w) * (kItems * 64) + k * 64 + lane;
        if (idx < P) {
            const uint32_t d = (key[k] >> shift) & (kRadix - 1);
            const uint32_t r = s_dstart[d] + s_wcnt[w][d] + loc[k];
            s_key[r] = K(key[k]);
            s_val[r] = val[k];
        }
    }
    __syncthreads();
    const int64_t nvalid = (P - base) < kTileKeys ? (P - base) : kTileKeys;
    for (int64_t j = t; j < nvalid; j += kSortThreads) {
        const K k = s_key[j];
        const uint32_t d = (uint32_t(k) >> shift) & (kRadix - 1);
        const int64_t pos = int64_t(s_gofs[d]) + (j - int64_t(s_dstart[d]));
        kout[pos] = k;
        vout[pos] = s_val[j];
        if constexpr (kRankCounts) {
            const uint4 r = recs_by_idx[s_val[j]];
            if (rank_counts) rank_counts[pos] = (static_cast<unsigned long long>(r.y) << 32) | r.x;
            rank_rects[pos] = (static_cast<unsigned long long>(r.w) << 32) | r.z;
        }
    }
}

// Up to this many Gaussians the depth sort takes 1024 keys per block instead of 4096: more, shorter
// blocks (the whole binning at 20k 109 -> 91 us, 60k 118 -> 106, 130k 127 -> 122; at 300k it is even,
// at 1M smaller tiles' longer look-back costs more: 201 -> 260).
constexpr int64_t kSort4 = 131072;
// Up to this many Gaussians one launch may write the lists, or one block place the entries (as many as are
// expected to be kSbOneEntries: two windows).
constexpr int kSmallSort = 4096;
constexpr double kSbOneEntries = 8192.0;

// The depth order of up to kRankSort Gaussians in one launch: a block ranks 64 of them (lane e) by
// counting the keys before theirs, a sixteenth of all per wavefront, four at a time from LDS (the same
// address for every lane). Two vector instructions per key and 64 Gaussians, n^2 / 64 of them in all;
// the passes' six launches wait for one another. Also k_bin_init's work. The whole binning of 2000
// Gaussians 45 -> 38 us (with four passes in one block's LDS before), of 8192 82 -> 63, 16384 87 -> 79;
// at 20000, where a second round of blocks begins, 90 -> 110.
constexpr int kRankSort = 16384, kRankThreads = 1024;
__global__ __launch_bounds__(kRankThreads) void k_rank(const float *depths, int n, uint32_t *sorted_idx,
                                                       const uint4 *recs_by_idx,
                                                       unsigned long long *rank_counts,
                                                       unsigned long long *rank_rects, uint32_t *ranges,
                                                       int ranges_n, SbTable *table, int32_t *status) {
    constexpr int kWaves = kRankThreads / 64;
    extern __shared__ __align__(16) uint32_t s_key[];        // n keys, to a multiple of 64
    __shared__ uint32_t s_part[kWaves][64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int e0 = int(blockIdx.x) * 64, e = e0 + lane, padded = (n + 63) & ~63;
    if (blockIdx.x == 0) {
        if (t < kSbLists) table->listed[t][0] = 0ull;
        if (t == 0) *status = GSB_OK;
    }
    for (int k = int(blockIdx.x) * kRankThreads + t; k < ranges_n; k += int(gridDim.x) * kRankThreads)
        ranges[k] = 0u;
    for (int i = t; i < padded; i += kRankThreads) s_key[i] = i < n ? depth_key(depths[i]) : ~0u;
    __syncthreads();
    const uint32_t my = s_key[e];
    const int part = (padded / kWaves + 3) & ~3;
    const int lo = w * part, hi = lo + part < padded ? lo + part : padded;
    uint32_t before = 0;
    const auto count = [&](int a, int b, auto test) {        // (a and b multiples of 4)
#pragma unroll 4
        for (int j = a; j < b; j += 4) {
            const uint4 k = *reinterpret_cast<const uint4 *>(&s_key[j]);
            before += test(k.x, j) ? 1u : 0u;
            before += test(k.y, j + 1) ? 1u : 0u;
            before += test(k.z, j + 2) ? 1u : 0u;
            before += test(k.w, j + 3) ? 1u : 0u;
        }
    };
    // equal depths keep the order of the indices
    count(lo, hi < e0 ? hi : e0, [&](uint32_t k, int) { return k <= my; });
    count(lo > e0 ? lo : e0, hi < e0 + 64 ? hi : e0 + 64,
          [&](uint32_t k, int j) { return k < my || (k == my && j < e); });
    count(lo > e0 + 64 ? lo : e0 + 64, hi, [&](uint32_t k, int) { return k < my; });
    s_part[w][lane] = before;
    __syncthreads();
    if (w != 0 || e >= n) return;
    uint32_t rank = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) rank += s_part[k][lane];
    const uint4 r = recs_by_idx[e];
    sorted_idx[rank] = uint32_t(e);
    if (rank_counts) rank_counts[rank] = (static_cast<unsigned long long>(r.y) << 32) | r.x;
    rank_rects[rank] = (static_cast<unsigned long long>(r.w) << 32) | r.z;
}

// Depth sort of the n Gaussians (count on the device): keys made from `depths`, values the
// indices, 4 chained passes; the last one also writes each Gaussian's pair count at its rank
// (rank_counts). The sorted indices end in va (4 passes, an even number).
template <int kItems>
void sort_depth(const float *depths, uint32_t *ka, uint32_t *kb, uint32_t *va, uint32_t *vb,
                const unsigned long long *count, int64_t n, SortState *st, uint32_t *lookback,
                int32_t *status, const uint4 *recs_by_idx, unsigned long long *rank_counts,
                unsigned long long *rank_rects, hipStream_t s) {
    constexpr int passes = 32 / kRadixBits;
    const int64_t nblk = sort_blocks(n, kItems);
    if (nblk == 0) return;
    const int64_t hb = nblk < kHistBlocks ? nblk : kHistBlocks;
    k_sort_hist<kItems><<<dim3(unsigned(hb)), kSortThreads, 0, s>>>(depths, ka, va, count, passes,
                                                                    st, lookback, nblk);
    uint32_t *kin = ka, *kout = kb, *vin = va, *vout = vb;
    for (int p = 0; p < passes; ++p) {
        const auto pass = p == passes - 1 ? k_radix_pass<true, true, uint32_t, kItems>
                                          : k_radix_pass<true, false, uint32_t, kItems>;
        pass<<<dim3(unsigned(nblk)), kSortThreads, 0, s>>>(
            kin, vin, kout, vout, count, p * kRadixBits, st->hist[p],
            lookback + int64_t(p) * nblk * kRadix, &st->ticket[p], status, nullptr, nblk, recs_by_idx,
            rank_counts, rank_rects);
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
}

// Tile sort of up to cap pairs (count on the device) on key bits [0, bits): per pass a per-block
// histogram, its exclusive scan and the scatter. (With thousands of tiles of keys the chained
// passes wait on long look-back chains; the three-step pass does not.) The data ends in (ka, va)
// after an even number of passes, in (kb, vb) after an odd one; returns the number of passes.
template <typename K>
int sort_tiles(K *ka, K *kb, uint32_t *va, uint32_t *vb, const unsigned long long *count,
               int64_t cap, int bits, uint32_t *hist, uint32_t *partial, int32_t *status,
               hipStream_t s) {
    const int64_t nblk = sort_blocks(cap);
    const int passes = (bits + kRadixBits - 1) / kRadixBits;
    if (nblk == 0) return passes;
    K *kin = ka, *kout = kb;
    uint32_t *vin = va, *vout = vb;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * kRadixBits;
        k_block_hist<<<dim3(unsigned(nblk)), kSortThreads, 0, s>>>(kin, count, shift, hist, nblk);
        launch_scan<uint32_t>(hist, int64_t(kRadix) * nblk, partial, nullptr, nullptr, s);
        k_radix_pass<false, false, K><<<dim3(unsigned(nblk)), kSortThreads, 0, s>>>(
            kin, vin, kout, vout, count, shift, nullptr, nullptr, nullptr, status, hist, nblk,
            nullptr, nullptr, nullptr);
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    return passes;
}

// ------------------------------------------------------------------------------- superblocks
// From the Gaussians in depth order to the tiles' lists by way of superblocks of 8 x 8 tiles
// (grids of at most kMaxSb of them, i.e. up to 65536 tiles):
//   1. k_sb_hist, scan, k_sb_scatter: each Gaussian's entry (its index and a 64-bit mask of the
//      superblock's tiles that it covers) goes to every superblock it touches, stably, so that a
//      superblock's entries are in rank order;
//   2. k_sb_count: the tiles' list lengths, by transposing the masks of 64 entries at a time
//      (64 x 64 bits over a wavefront: lane t then holds which entries cover tile t);
//   3. k_tile_scan: the tiles' ranges;
//   4. k_sb_write: the transposed masks again, and the lists, assembled in LDS and written out in
//      runs of one tile each.
// The work per pair is the lane's own step through its set bits and one write of the list, half a
// vector instruction per pair, where a radix sort of the pairs takes about 2.3 per pass for ranking
// alone, two passes, and reads and writes every pair in each. (A Gaussian touches 18 tiles but only
// 1.6 superblocks on the 4K frame of 3M Gaussians, so what is sorted is a tenth.) Measured at 4K,
// 54.7M pairs, from the sorted Gaussians to the ranges: 0.18 ms against 0.84. In mode 1 the masks hold
// the visible tiles alone: 0.33 ms against 0.50.
constexpr int kSbMaxGrid = 4096;                         // blocks of steps 2 and 4, which loop
constexpr int kSbStage = 2 * kSbTiles * 64;              // pairs assembled in LDS at a time

struct SbGrid {
    int32_t gx, gy, sx, n;          // tile columns and rows, superblock columns, superblocks
};
__host__ __device__ inline SbGrid sb_grid(int32_t gx, int32_t gy) {
    const int32_t sx = (gx + kSbEdge - 1) >> kSbShift, sy = (gy + kSbEdge - 1) >> kSbShift;
    return SbGrid{gx, gy, sx, sx * sy};
}
// Entries per Gaussian to expect of `cap` pairs of n: a square of that many tiles, anywhere.
inline double sb_entries(int64_t n, int64_t cap) {
    const double side = sqrt(double(cap) / double(n)) / kSbEdge + 1.0;
    return side * side;
}
// Ranks per block of step 1. The digit counts (superblocks x blocks) take the place of the depth sort's
// look-back words (256 per 1024 Gaussians): 1024 to 4096 always fit. Of Gaussians of more than 64 tiles
// (about four entries) as many as one window of entries is expected of, if the counts have room, which
// grows with the pairs: with 1024 and more, a few blocks had all the entries of large Gaussians (the
// whole binning at 4K: 4000 Gaussians of 1000 px 124 ms, now 0.31, of 100 px 3.7 ms, now 0.11; 16384 of 100
// px 1.56 ms, now 0.16; 5000 of 1000 px in mode 1 58 ms, now 25).
inline int sb_ranks(int32_t n_sb, int64_t n, int64_t cap) {
    int ranks = n_sb <= 256 ? 1024 : n_sb <= 512 ? 2048 : 4096;
    if (cap / 64 <= n) return ranks;
    const double want = 4096.0 / sb_entries(n, cap);
    const int64_t words = sort_words(n, cap), room = words < kScanMaxLen ? words : kScanMaxLen;
    while (ranks > 8 && ranks > want && int64_t(n_sb) * ((2 * n + ranks - 1) / ranks + 1) <= room) ranks /= 2;
    return ranks;
}
// The superblock path where it applies: a grid of at most kMaxSb superblocks
inline bool by_superblock(const SbGrid &G) { return G.n <= kMaxSb; }

// Superblocks touched by a (non-empty) tile rectangle
__device__ inline Rect sb_rect(const Rect &R) {
    return Rect{R.tx0 >> kSbShift, (R.tx1 + kSbEdge - 1) >> kSbShift, R.ty0 >> kSbShift,
                (R.ty1 + kSbEdge - 1) >> kSbShift};
}
// Tiles [a - 8 s, b - 8 s) of superblock s along one axis, as a byte ([a, b) meets the superblock)
__device__ inline uint32_t sb_span(int a, int b, int s) {
    const int lo = a - s * kSbEdge, hi = (s + 1) * kSbEdge - b;
    return (0xffu >> (hi > 0 ? hi : 0)) & (0xffu << (lo > 0 ? lo : 0)) & 0xffu;
}
// The mask of a superblock's tiles, bit 8 row + column, from its columns (byte 0) and rows (byte 1)
__device__ inline unsigned long long sb_mask(uint32_t clip) {
    const uint32_t cols = (clip & 0xffu) * 0x01010101u, rows = clip >> 8;
    // each of four rows as a byte of ones: the row's bit spread to its byte's bit 0, times 255
    const uint32_t lo = ((rows & 0xfu) * 0x00204081u) & 0x01010101u;
    const uint32_t hi = ((rows >> 4) * 0x00204081u) & 0x01010101u;
    return (unsigned long long)(cols & (lo * 255u)) | ((unsigned long long)(cols & (hi * 255u)) << 32);
}

__global__ __launch_bounds__(kSortThreads) void k_sb_hist(const unsigned long long *rank_rects,
                                                          int64_t n, int ranks, SbGrid G,
                                                          uint32_t *hist, int64_t nblk) {
    __shared__ uint32_t s_h[kMaxSb];
    const int t = threadIdx.x;
    for (int d = t; d < G.n; d += kSortThreads) s_h[d] = 0u;
    __syncthreads();
    const int64_t blk = xcd_rank(blockIdx.x, uint32_t(nblk));
    if (blk >= nblk) return;                                 // block-uniform
    const int64_t j0 = blk * ranks;
    for (int k = t; k < ranks; k += kSortThreads) {
        if (j0 + k >= n) break;
        const Rect R = unpack_rect(rank_rects[j0 + k]);
        if (R.tx1 <= R.tx0 || R.ty1 <= R.ty0) continue;
        const Rect Q = sb_rect(R);
        for (int sy = Q.ty0; sy < Q.ty1; ++sy)
            for (int sx = Q.tx0; sx < Q.tx1; ++sx) atomicAdd(&s_h[sy * G.sx + sx], 1u);
    }
    __syncthreads();
    for (int d = t; d < G.n; d += kSortThreads) hist[int64_t(d) * nblk + blk] = s_h[d];
}

// Mode 1: the tiles of superblock (sx, sy) that are visible, from the candidates' mask (sb_form).
__device__ inline unsigned long long sb_submask(const Rect &R, unsigned long long mask, int sx, int sy) {
    const int dx = R.tx0 - sx * kSbEdge, dy = R.ty0 - sy * kSbEdge;       // within +-7
    mask = dy >= 0 ? mask << (8 * dy) : mask >> (-8 * dy);
    mask = dx >= 0 ? mask << dx : mask >> -dx;
    const uint32_t cols = ((dx >= 0 ? 0xffu << dx : 0xffu >> -dx) & 0xffu) * 0x01010101u;
    return mask & ((static_cast<unsigned long long>(cols) << 32) | cols);
}

// Mode 1: the superblocks with a visible tile. Those of a rectangle that its candidate mask covers are
// cut from it. Those of a larger one are listed by k_sb_list, from the end of the entries' arrays
// downwards; a Gaussian's record holds its place and their number << 48. There are `lists` lists, in
// alternate runs of kSbListRun places: with one counter for all, the XCDs' atomics on it took 400 us
// of 3 M Gaussians (20 ns each). The masks are tested again where the arrays had no room for them,
// which takes more than one such superblock for two pairs (a thin line has 8 pairs in each).
struct SbVisible {
    const unsigned long long *rank_masks;
    uint4 *recs;
    unsigned long long *masks;                    // the arrays' ends: place o is [-1 - o]
    uint32_t *sbs;
    const SbTable *table;
    int lists;                                    // a power of two
    const float2 *means;
    const float *conics, *opac;
    int32_t W, H;
};
__device__ inline unsigned long long sb_test(const SbVisible &V, const Rect &R, uint32_t i, int sx, int sy) {
    const Vis32 g = vis32_setup(V.means[i], V.conics + 3 * int64_t(i), V.opac[i], nullptr, R);
    unsigned long long m = 0;
#pragma unroll 1
    for (int b = 0; b < kSbTiles; ++b) {
        const int tx = sx * kSbEdge + (b & (kSbEdge - 1)), ty = sy * kSbEdge + (b >> kSbShift);
        if (tx >= R.tx0 && tx < R.tx1 && ty >= R.ty0 && ty < R.ty1 && tile_visible(g, tx, ty, V.W, V.H))
            m |= 1ull << b;
    }
    return m;
}
// the places of list `l`'s entries
__device__ inline unsigned long long sb_place(unsigned long long o, int l, int lists) {
    return (o / kSbListRun * lists + l) * kSbListRun + o % kSbListRun;
}
__device__ inline unsigned long long sb_listed(const SbVisible &V) {      // places up to the last
    unsigned long long most = 0;
    for (int l = 0; l < V.lists; ++l) {
        const unsigned long long e = V.table->listed[l][0];
        most = e > most ? e : most;
    }
    return sb_place(most + kSbListRun - 1, 0, V.lists) / kSbListRun * kSbListRun;
}
// f(superblock, mask) for every superblock of Gaussian *i with a visible tile.
template <class F>
__device__ inline void sb_visible(const SbVisible &V, const SbGrid &G, const Rect &R,
                                  unsigned long long mask, const uint32_t *i, bool listed,
                                  F f) {
    if (R.tx1 <= R.tx0 || R.ty1 <= R.ty0) return;
    const bool big = sb_big(R);
    if (big && listed) {
        const uint2 r = reinterpret_cast<const uint2 *>(V.recs + *i)[0];
        mask = (static_cast<unsigned long long>(r.y) << 32) | r.x;
        const unsigned long long o = mask & ((1ull << 45) - 1ull);
        const int l = int(mask >> 45) & 7, e = int(mask >> 48);
#pragma unroll 1
        for (int k = 0; k < e; k += 4) {                     // four loads at a time (99 us, now 89)
            uint32_t sb[4];
            unsigned long long m[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t p = int64_t(sb_place(o + (k + q < e ? k + q : k), l, V.lists));
                sb[q] = V.sbs[-1 - p];
                m[q] = V.masks[-1 - p];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k + q < e) f(sb[q], m[q]);
        }
        return;
    }
    const Rect q = sb_rect(R);
#pragma unroll 1
    for (int sy = q.ty0; sy < q.ty1; ++sy)
#pragma unroll 1
        for (int sx = q.tx0; sx < q.tx1; ++sx) {
            const unsigned long long m = big ? sb_test(V, R, *i, sx, sy) : sb_submask(R, mask, sx, sy);
            if (m != 0ull) f(uint32_t(sy * G.sx + sx), m);
        }
}

// The list of the Gaussians with candidates past a mask's 8 x 8, each tested by a whole wavefront,
// a superblock's 64 tiles at a time. In the order of the indices, as large Gaussians are neighbours
// in the order of depth. Masks are gathered in LDS, for an atomic per kMaxSb of them or wavefront. A
// wavefront takes eight at a time (a cache line of records) from all over the indices, so that a run of
// large ones is not one wavefront's (64 of 1500 px in a row at 4K: 5.9 ms, now 0.74).
__global__ __launch_bounds__(64, 5) void k_sb_list(SbVisible V, SbTable *table,
                                                int64_t n, SbGrid G, int64_t cap) {
    __shared__ unsigned long long s_mask[kMaxSb];
    __shared__ uint16_t s_sb[kMaxSb];
    const int lane = threadIdx.x, l = int(blockIdx.x) & (V.lists - 1);    // (an XCD's own list)
    const int64_t i = (int64_t(lane >> 3) * gridDim.x + blockIdx.x) * 8 + (lane & 7);
    Rect R{0, 0, 0, 0};
    if (i < n) {
        const uint2 z = reinterpret_cast<const uint2 *>(V.recs + i)[1];
        R = unpack_rect((static_cast<unsigned long long>(z.y) << 32) | z.x);
    }
    const bool big = R.tx1 > R.tx0 && R.ty1 > R.ty0 && sb_big(R);
    unsigned long long todo = __ballot(big);
    if (todo == 0ull) return;                                // wavefront-uniform
    const Rect Q = big ? sb_rect(R) : Rect{0, 0, 0, 0};
    Vis32 own{};
    if (big) own = vis32_setup(V.means[i], V.conics + 3 * i, V.opac[i], nullptr, R);
    int fill = 0;                                            // masks in LDS (uniform)
    int place = 0, mine = 0;                                 // this lane's: the first and how many
    bool waits = false;
    const auto flush = [&] {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(&table->listed[l][0], (unsigned long long)fill);
        base = __shfl(base, 0, 64);
        if (waits) {
            const unsigned long long r = (base + place) | ((unsigned long long)(l | mine << 3) << 45);
            reinterpret_cast<uint2 *>(V.recs + i)[0] = make_uint2(uint32_t(r), uint32_t(r >> 32));
        }
        waits = false;
        __builtin_amdgcn_wave_barrier();
        for (int k = lane; k < fill; k += 64) {
            const int64_t o = int64_t(sb_place(base + k, l, V.lists));
            if (o < cap) {
                V.masks[-1 - o] = s_mask[k];
                V.sbs[-1 - o] = s_sb[k];
            }
        }
        __builtin_amdgcn_wave_barrier();
        fill = 0;
    };
    while (todo) {
        const int src = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        const auto from = [&](int v) { return __builtin_amdgcn_readlane(v, src); };
        const Rect S{from(R.tx0), from(R.tx1), from(R.ty0), from(R.ty1)};
        const Rect P{from(Q.tx0), from(Q.tx1), from(Q.ty0), from(Q.ty1)};
        const auto fromf = [&](float v) { return __int_as_float(from(__float_as_int(v))); };
        const Vis32 g{fromf(own.x), fromf(own.y), fromf(own.A), fromf(own.B), fromf(own.C),
                      fromf(own.o), fromf(own.rA), fromf(own.rC), fromf(own.lo), fromf(own.hi)};
        if (fill + (P.tx1 - P.tx0) * (P.ty1 - P.ty0) > kMaxSb) flush();
        const int first = fill;
        for (int sy = P.ty0; sy < P.ty1; ++sy)
            for (int sx = P.tx0; sx < P.tx1; ++sx) {
                const int tx = sx * kSbEdge + (lane & (kSbEdge - 1)), ty = sy * kSbEdge + (lane >> kSbShift);
                const bool v = tx >= S.tx0 && tx < S.tx1 && ty >= S.ty0 && ty < S.ty1 &&
                               tile_visible(g, tx, ty, V.W, V.H);
                const unsigned long long m = __ballot(v);
                if (m == 0ull) continue;
                if (lane == 0) {
                    s_mask[fill] = m;
                    s_sb[fill] = uint16_t(sy * G.sx + sx);
                }
                ++fill;
            }
        if (lane == src) {
            place = first;
            mine = fill - first;
            waits = true;
        }
    }
    flush();
}

// A Gaussian with more than kSbSerial entries in a window of k_sb_scatter is listed in LDS there, and a
// wavefront writes them, an entry per lane: by their owner alone, a window of Gaussians of 500 entries
// took 230 us. Blocks without one (all but a few on usual frames, whose largest have 16 to 25) skip the
// listing's barriers.
constexpr int kSbSerial = 32;

// Mode 1: as k_sb_hist, for the superblocks with a visible tile; also the place of each rank's first
// entry among its block's, and the number of the block's (with kSbMany: a rank has more than kSbSerial).
constexpr uint32_t kSbMany = 1u << 31;
__global__ __launch_bounds__(kSortThreads, 6) void k_sb_hist_visible(
    const unsigned long long *rank_rects, const uint32_t *sorted_idx, SbVisible V, int64_t n, int ranks,
    SbGrid G, uint32_t *hist, int64_t nblk, int64_t cap, uint32_t *rank_pos,
    uint32_t *block_entries) {
    __shared__ uint32_t s_h[kMaxSb], s_wave[kSortThreads / 64], s_many;
    const int t = threadIdx.x;
    for (int d = t; d < G.n; d += kSortThreads) s_h[d] = 0u;
    if (t == 0) s_many = 0u;
    __syncthreads();
    const int64_t blk = xcd_rank(blockIdx.x, uint32_t(nblk));
    if (blk >= nblk) return;                                 // block-uniform
    const bool listed = sb_listed(V) <= (unsigned long long)cap;
    const int64_t j0 = blk * ranks;
    uint32_t first = 0;
    unsigned long long rect = 0, mask = 0, next_rect = 0, next_mask = 0;   // loaded a step ahead
    const int64_t end = n - j0 < ranks ? n : j0 + ranks;
    const auto load = [&](int64_t j) {
        next_rect = next_mask = 0;
        if (j < end) {
            next_rect = rank_rects[j];
            next_mask = V.rank_masks[j];
        }
    };
    load(j0 + t);
    for (int k = 0; j0 + k < end; k += kSortThreads) {                  // block-uniform
        const int64_t j = j0 + k + t;
        uint32_t e = 0, step;
        rect = next_rect;
        mask = next_mask;
        load(j + kSortThreads);
        if (j < end)
            sb_visible(V, G, unpack_rect(rect), mask, sorted_idx + j, listed,
                       [&](uint32_t sb, unsigned long long) {
                           atomicAdd(&s_h[sb], 1u);
                           ++e;
                       });
        if (e > uint32_t(kSbSerial)) s_many = kSbMany;
        const uint32_t pos = block_exclusive_scan<uint32_t>(e, s_wave, step);
        if (j < end) rank_pos[j] = first + pos;
        first += step;
    }
    __syncthreads();
    if (t == 0) block_entries[blk] = first | s_many;
    for (int d = t; d < G.n; d += kSortThreads) hist[int64_t(d) * nblk + blk] = s_h[d];
}

// A block places the entries of its ranks: thread t owns kPer consecutive ones, whose rectangles and
// indices it loads first, all at once (a load per rank in the loop over ranks left two blocks per
// CU waiting: 107 us at 4K, now 61). The block's entries, enumerated in rank order, are taken
// kSbWindow at a time: written to LDS by their owners, ranked within their superblock as in
// k_radix_pass, reordered in LDS and written out in runs. The blocks of one XCD take consecutive
// ranks (xcd_rank): a superblock's entries from neighbouring blocks are neighbours in memory, a run
// is shorter than a cache line, and the line is put together in that XCD's L2 (12% less time).
// Block 0 also fills the superblock table. kOne: the only block (nblk = 1) counts its entries per
// superblock itself, with no launches of k_sb_hist and its scan. kVis: mode 1, entries with a visible
// tile and their masks (half the window, as masks do not fit the keys' spare bits).
template <int kPer, bool kOne, bool kVis>
__global__ __launch_bounds__(kSortThreads) void k_sb_scatter(
    const unsigned long long *rank_rects, const uint32_t *sorted_idx, int64_t n, int ranks, SbGrid G, int bits,
    const uint32_t *hist, int64_t nblk, BinHeader *hdr, int64_t cap, uint32_t chunk, uint32_t *e_idx,
    unsigned long long *e_mask, SbTable *table, SbVisible V,
    const uint32_t *rank_pos, const uint32_t *block_entries) {
    static_assert(!(kOne && kVis), "mode 1 counts in k_sb_hist_visible");
    constexpr int kSbWindow = kVis ? 2048 : 4096, kSbSteps = kSbWindow / kSortThreads;
    constexpr int kWaves = kSortThreads / 64, kDig = kMaxSb / kSortThreads;
    __shared__ uint32_t s_gofs[kMaxSb];                 // next global position of each superblock
    // per-wave counts, then prefixes; before that the window's listed ranks (rectangle, or mode 1 the
    // masks' place; index; first entry, from the window's start)
    __shared__ __align__(16) uint16_t s_wcnt[kWaves][kMaxSb];
    uint4 *const s_list = reinterpret_cast<uint4 *>(&s_wcnt[0][0]);
    static_assert(sizeof(s_wcnt) / sizeof(uint4) > kSbWindow / (kSbSerial + 1), "a place for each listed rank");
    __shared__ int s_listed;
    __shared__ uint32_t s_large[kWaves];                // a rank of the wavefront has many entries
    __shared__ uint16_t s_dstart[kMaxSb];               // start of each superblock in the window
    __shared__ uint32_t s_wave[kWaves];
    __shared__ uint32_t s_key[kSbWindow];               // superblock | columns << 16 | rows << 24
    __shared__ uint32_t s_idx[kSbWindow];
    __shared__ unsigned long long s_mask[kVis ? kSbWindow : 1];
    __shared__ int s_rank;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t blk = xcd_rank(blockIdx.x, uint32_t(nblk));
    if (blk >= nblk) return;                                 // block-uniform
    // this thread's ranks: superblocks (0 x 0 where the rectangle is empty or past the end),
    // rectangle and index. kPer is a multiple of 4 and the buffers are padded to 256 bytes, so the
    // vector loads that straddle n stay inside them.
    // (`ranks` is a multiple of kPer, at most kPer per thread.)
    const int64_t j0 = blk * ranks + int64_t(t) * kPer;
    const int64_t n_own = t * kPer < ranks ? n : 0;          // past the block's ranks: none
    unsigned long long rects[kPer];
    uint32_t idx[kPer], mine = 0;
    // (loaded again for a second window: kept through the first, their registers cost a block per CU)
    const auto load_ranks = [&] {
        if constexpr (kPer == 1) {
            rects[0] = j0 < n_own ? rank_rects[j0] : 0ull;
            idx[0] = j0 < n_own ? sorted_idx[j0] : 0u;
        }
#pragma unroll
        for (int k = 0; k < (kPer == 1 ? 0 : kPer); k += 4) {
            ulonglong2 r01{0, 0}, r23{0, 0};
            uint4 i4{0, 0, 0, 0};
            if (j0 + k < n_own) {
                r01 = *reinterpret_cast<const ulonglong2 *>(rank_rects + j0 + k);
                i4 = *reinterpret_cast<const uint4 *>(sorted_idx + j0 + k);
            }
            if (j0 + k + 2 < n_own) r23 = *reinterpret_cast<const ulonglong2 *>(rank_rects + j0 + k + 2);
            rects[k] = r01.x;
            rects[k + 1] = j0 + k + 1 < n_own ? r01.y : 0;
            rects[k + 2] = r23.x;
            rects[k + 3] = j0 + k + 3 < n_own ? r23.y : 0;
            idx[k] = i4.x; idx[k + 1] = i4.y; idx[k + 2] = i4.z; idx[k + 3] = i4.w;
        }
    };
    if constexpr (!kVis) load_ranks();
    const auto entries = [](const Rect &r) {
        if (r.tx1 <= r.tx0 || r.ty1 <= r.ty0) return 0u;
        const Rect q = sb_rect(r);
        return uint32_t((q.tx1 - q.tx0) * (q.ty1 - q.ty0));
    };
    bool large = false;
    if constexpr (!kVis) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const uint32_t e = entries(unpack_rect(rects[k]));
            mine += e;
            large = large || e > uint32_t(kSbSerial);
        }
        const bool any = __ballot(large) != 0ull;
        if (lane == 0) s_large[w] = any ? 1u : 0u;           // (read behind the scan's barriers)
    }
    uint32_t n_entries;
    if constexpr (kOne) {
        for (int d = t; d < kMaxSb; d += kSortThreads) s_gofs[d] = 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const Rect R = unpack_rect(rects[k]);
            if (entries(R) == 0u) continue;
            const Rect q = sb_rect(R);
            for (int sy = q.ty0; sy < q.ty1; ++sy)
                for (int sx = q.tx0; sx < q.tx1; ++sx) atomicAdd(&s_gofs[sy * G.sx + sx], 1u);
        }
        __syncthreads();
        uint32_t c[kDig], sum = 0;
#pragma unroll
        for (int q = 0; q < kDig; ++q) sum += c[q] = s_gofs[t * kDig + q];
        uint32_t run = block_exclusive_scan<uint32_t>(sum, s_wave, n_entries);
#pragma unroll
        for (int q = 0; q < kDig; ++q) {
            s_gofs[t * kDig + q] = run;
            run += c[q];
        }
        __syncthreads();
    } else {
        for (int d = t; d < G.n; d += kSortThreads) s_gofs[d] = hist[int64_t(d) * nblk + blk];
        n_entries = uint32_t(hdr->entries);
    }
    if (blk == 0) {
        // four superblocks per thread: starts from the scanned counts, chunks from their sizes.
        // No entries at all when the pairs exceed the capacity (every list is then empty); else
        // there are at most as many entries as pairs.
        const uint32_t total = hdr->total <= (unsigned long long)cap ? n_entries : 0u;
        uint32_t st[kDig + 1], ch[kDig], sum = 0, tot;
#pragma unroll
        for (int k = 0; k <= kDig; ++k) {
            const int d = t * kDig + k;
            const uint32_t v = d < G.n ? (kOne ? s_gofs[d] : hist[int64_t(d) * nblk]) : total;
            st[k] = v < total ? v : total;              // (entries past the capacity do not exist)
        }
#pragma unroll
        for (int k = 0; k < kDig; ++k) {
            ch[k] = (st[k + 1] - st[k] + chunk - 1) / chunk;
            sum += ch[k];
        }
        uint32_t run = block_exclusive_scan<uint32_t>(sum, s_wave, tot);
#pragma unroll
        for (int k = 0; k < kDig; ++k) {
            table->start[t * kDig + k] = st[k];
            table->chunk[t * kDig + k] = run;
            run += ch[k];
        }
        if (t == kSortThreads - 1) {
            table->start[kMaxSb] = total;
            table->chunk[kMaxSb] = run;
        }
    }
    if (kVis && hdr->total > (unsigned long long)cap) return;   // block-uniform; every list is empty
    uint32_t total = 0, pos0 = 0;
    if constexpr (kVis) {
        total = block_entries[blk];
        large = (total & kSbMany) != 0u;
        total &= kSbMany - 1u;
    } else {
        pos0 = block_exclusive_scan<uint32_t>(mine, s_wave, total);
        large = (s_large[0] | s_large[1] | s_large[2] | s_large[3]) != 0u;
    }
    const uint32_t serial = large ? uint32_t(kSbSerial) : ~0u;
    for (uint32_t w0 = 0; w0 < total; w0 += kSbWindow) {      // block-uniform
        const int cnt = int(total - w0 < uint32_t(kSbWindow) ? total - w0 : uint32_t(kSbWindow));
        [[maybe_unused]] uint32_t pos = pos0;
        // the part [lo, hi) of a rank's entries [pos, pos + e) that lies in the window
        [[maybe_unused]] const auto part = [&](uint32_t e, uint32_t &lo, uint32_t &hi) {
            lo = pos < w0 ? w0 - pos : 0u;
            hi = pos >= w0 + kSbWindow ? 0u : e < w0 + kSbWindow - pos ? e : w0 + kSbWindow - pos;
        };
        if constexpr (kVis) {
            // rank k kSortThreads + t of the block, the next one's data loaded ahead
            const bool listed = sb_listed(V) + hdr->entries <= (unsigned long long)cap;
            const int64_t b0 = blk * ranks;
            const int own = int(n - b0 < ranks ? n - b0 : ranks);
            struct Rank {
                uint32_t pos, end, idx;
                unsigned long long rect, mask;
            };
            const auto load = [&](int r) {
                Rank a{total, total, 0, 0, 0};
                if (r < own) {
                    a.pos = rank_pos[b0 + r];
                    if (r + 1 < own) a.end = rank_pos[b0 + r + 1];
                    a.idx = sorted_idx[b0 + r];
                    a.rect = rank_rects[b0 + r];
                    a.mask = V.rank_masks[b0 + r];
                }
                return a;
            };
            const int r0 = w0 > 0 ? s_rank : 0;              // the window's first rank
            Rank next = load(r0 + t);
            if (large && t == 0) s_listed = 0;
            if (large || w0 > 0) __syncthreads();            // s_rank has been read
#pragma unroll 1
            for (int r = r0 + t; r < own; r += kSortThreads) {
                const Rank a = next;
                if (a.pos >= w0 + kSbWindow) break;
                next = load(r + kSortThreads);
                if (a.end >= w0 + kSbWindow) s_rank = r;     // the last rank that starts here
                if (a.end <= w0 || a.pos == a.end) continue;
                uint32_t o = a.pos - w0;                 // (wraps while before the window)
                const uint32_t lo = a.pos > w0 ? a.pos : w0;
                const uint32_t hi = a.end < w0 + kSbWindow ? a.end : w0 + kSbWindow;
                if (large && listed && hi - lo > uint32_t(kSbSerial) && sb_big(unpack_rect(a.rect))) {
                    const uint2 p = reinterpret_cast<const uint2 *>(V.recs + a.idx)[0];
                    s_list[atomicAdd(&s_listed, 1)] = make_uint4(p.x, p.y, a.idx, o);
                    continue;
                }
                sb_visible(V, G, unpack_rect(a.rect), a.mask, &a.idx, listed,
                           [&](uint32_t sb, unsigned long long m) {
                               if (o < uint32_t(kSbWindow)) {
                                   s_key[o] = sb;
                                   s_idx[o] = a.idx;
                                   s_mask[o] = m;
                               }
                               ++o;
                           });
            }
            if (large) {                                     // block-uniform
                __syncthreads();
                const int listed_n = s_listed;
                for (int i = w; i < listed_n; i += kWaves) {
                    const uint4 q = s_list[i];
                    const unsigned long long p = (static_cast<unsigned long long>(q.y) << 32) | q.x;
                    const unsigned long long place = p & ((1ull << 45) - 1ull);
                    const int l = int(p >> 45) & 7, e = int(p >> 48), first = int(q.w);
                    const int last = first + e < kSbWindow ? first + e : kSbWindow;
                    for (int o = (first > 0 ? first : 0) + lane; o < last; o += 64) {
                        const int64_t at = int64_t(sb_place(place + (o - first), l, V.lists));
                        s_key[o] = V.sbs[-1 - at];
                        s_mask[o] = V.masks[-1 - at];
                        s_idx[o] = q.z;
                    }
                }
                __syncthreads();                             // before the counts take the list's place
            }
        } else {
            if (w0 > 0) load_ranks();
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const Rect R = unpack_rect(rects[k]);
                const uint32_t e = entries(R);
                uint32_t lo, hi;
                part(e, lo, hi);
                if (lo < hi && hi - lo <= serial) {
                    const Rect q = sb_rect(R);
                    const uint32_t wd = uint32_t(q.tx1 - q.tx0);
                    int sy = q.ty0, sx = q.tx0;
                    if (lo > 0) {
                        sy += int(lo / wd);
                        sx += int(lo % wd);
                    }
                    uint32_t row = uint32_t(sy * G.sx) | (sb_span(R.ty0, R.ty1, sy) << 24);
                    for (uint32_t o = pos + lo - w0; o < pos + hi - w0; ++o) {
                        s_key[o] = (row + uint32_t(sx)) | (sb_span(R.tx0, R.tx1, sx) << 16);
                        s_idx[o] = idx[k];
                        if (++sx == q.tx1) {
                            sx = q.tx0;
                            ++sy;
                            row = uint32_t(sy * G.sx) | (sb_span(R.ty0, R.ty1, sy) << 24);
                        }
                    }
                }
                pos += e;
            }
            if (large) {                                     // block-uniform
                if (t == 0) s_listed = 0;
                __syncthreads();
                // (the ranks are loaded again: held for this, their registers cost a block per CU)
                pos = pos0;
#pragma unroll 1
                for (int k = 0; k < kPer && j0 + k < n_own; ++k) {
                    const unsigned long long rect = rank_rects[j0 + k];
                    const uint32_t e = entries(unpack_rect(rect));
                    uint32_t lo, hi;
                    part(e, lo, hi);
                    if (lo < hi && hi - lo > serial)
                        s_list[atomicAdd(&s_listed, 1)] = make_uint4(uint32_t(rect), uint32_t(rect >> 32),
                                                                     sorted_idx[j0 + k], pos - w0);
                    pos += e;
                }
                __syncthreads();
                const int listed_n = s_listed;
                for (int i = w; i < listed_n; i += kWaves) {
                    const uint4 p = s_list[i];
                    const Rect R = unpack_rect((static_cast<unsigned long long>(p.y) << 32) | p.x);
                    const Rect q = sb_rect(R);
                    const int wd = q.tx1 - q.tx0, e = wd * (q.ty1 - q.ty0), first = int(p.w);
                    const int last = first + e < kSbWindow ? first + e : kSbWindow;
                    for (int o = (first > 0 ? first : 0) + lane; o < last; o += 64) {
                        const int sy = q.ty0 + (o - first) / wd, sx = q.tx0 + (o - first) % wd;
                        s_key[o] = uint32_t(sy * G.sx + sx) | (sb_span(R.tx0, R.tx1, sx) << 16) |
                                   (sb_span(R.ty0, R.ty1, sy) << 24);
                        s_idx[o] = p.z;
                    }
                }
                __syncthreads();                             // before the counts take the list's place
            }
        }
        for (int d = t; d < kMaxSb; d += kSortThreads) {
#pragma unroll
            for (int i = 0; i < kWaves; ++i) s_wcnt[i][d] = 0;
        }
        __syncthreads();
        // wave w ranks the entries [w seg, (w + 1) seg) of the window, 64 at a time
        const int steps = (cnt + kSortThreads - 1) / kSortThreads, seg = steps * 64;
        uint32_t key[kSbSteps], loc[kSbSteps], id[kSbSteps];
        unsigned long long mk[kVis ? kSbSteps : 1];
#pragma unroll
        for (int i = 0; i < kSbSteps; ++i) {
            if (i >= steps) break;                           // uniform
            const int o = w * seg + i * 64 + lane;
            const bool valid = o < cnt;
            const int oc = valid ? o : 0;
            key[i] = s_key[oc];
            id[i] = s_idx[oc];
            if constexpr (kVis) mk[i] = s_mask[oc];
            const uint32_t d = key[i] & 0xffffu;
            const unsigned long long vmask = __builtin_amdgcn_ballot_w64(valid);
            uint32_t plo = uint32_t(vmask), phi = uint32_t(vmask >> 32);
            const uint32_t nd = ~d;
#pragma unroll
            for (int b = 0; b < kMaxSbBits; ++b) {
                if (b >= bits) break;                        // uniform
                const uint32_t flip = uint32_t(int32_t(nd << (31 - b)) >> 31);
                const unsigned long long vote = __builtin_amdgcn_ballot_w64(flip == 0u);
                plo &= uint32_t(vote) ^ flip;
                phi &= uint32_t(vote >> 32) ^ flip;
            }
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
            uint32_t prior = 0;
            if (valid) prior = s_wcnt[w][d];
            if (valid && rank == 0)
                s_wcnt[w][d] = uint16_t(prior + uint32_t(__popc(plo) + __popc(phi)));
            loc[i] = prior + rank;
        }
        __syncthreads();
        // thread t: superblocks 4t .. 4t + 3, exclusive prefix over waves and the window's starts
        uint32_t c[kDig], sum = 0, tot;
#pragma unroll
        for (int q = 0; q < kDig; ++q) {
            uint32_t run = 0;
#pragma unroll
            for (int i = 0; i < kWaves; ++i) {
                const uint32_t v = s_wcnt[i][t * kDig + q];
                s_wcnt[i][t * kDig + q] = uint16_t(run);
                run += v;
            }
            c[q] = run;
            sum += run;
        }
        uint32_t run = block_exclusive_scan<uint32_t>(sum, s_wave, tot);
#pragma unroll
        for (int q = 0; q < kDig; ++q) {
            s_dstart[t * kDig + q] = uint16_t(run);
            run += c[q];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSbSteps; ++i) {
            if (i >= steps) break;
            if (w * seg + i * 64 + lane < cnt) {
                const uint32_t d = key[i] & 0xffffu, r = s_dstart[d] + s_wcnt[w][d] + loc[i];
                s_key[r] = key[i];
                s_idx[r] = id[i];
                if constexpr (kVis) s_mask[r] = mk[i];
            }
        }
        __syncthreads();
        for (int o = t; o < cnt; o += kSortThreads) {
            const uint32_t key_o = s_key[o], d = key_o & 0xffffu;
            const int64_t p = int64_t(s_gofs[d]) + (o - int(s_dstart[d]));
            if (p < cap) {
                e_idx[p] = s_idx[o];
                e_mask[p] = kVis ? s_mask[kVis ? o : 0] : sb_mask(key_o >> 16);
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kDig; ++q) s_gofs[t * kDig + q] += c[q];
        __syncthreads();
    }
}

// The 64 x 64 bit matrix whose row l is lane l's m, transposed: lane t gets bit t of every row.
// Each level exchanges a block of columns with the lane whose index differs in that bit.
__device__ inline unsigned long long transpose64(unsigned long long m, int lane) {
    uint32_t v[2];
    {
        const auto r = __builtin_amdgcn_permlane32_swap(uint32_t(m), uint32_t(m >> 32), false, false);
        v[0] = r[0];
        v[1] = r[1];
    }
    // bytes of (own, partner) kept on each side of the 16- and 8-lane exchanges
    const uint32_t sel16 = (lane & 16) ? 0x07060302u : 0x05040100u;
    const uint32_t sel8 = (lane & 8) ? 0x03070105u : 0x06020400u;
    const uint32_t rot4 = (lane & 4) ? 4 : 28, keep4 = (lane & 4) ? 0xf0f0f0f0u : 0x0f0f0f0fu;
    const uint32_t rot2 = (lane & 2) ? 2 : 30, keep2 = (lane & 2) ? 0xccccccccu : 0x33333333u;
    const uint32_t rot1 = (lane & 1) ? 1 : 31, keep1 = (lane & 1) ? 0xaaaaaaaau : 0x55555555u;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(v[i], v[i], false, false);
        uint32_t x = __builtin_amdgcn_perm(r[1], r[0], sel16);
        uint32_t y = uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x128, 0xf, 0xf, true));
        x = __builtin_amdgcn_perm(y, x, sel8);
        // lane ^ 4 = (7 - lane) ^ 3 within 8 lanes
        y = uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x141, 0xf, 0xf, true));
        y = uint32_t(__builtin_amdgcn_update_dpp(0, int(y), 0x1b, 0xf, 0xf, true));
        x = (x & keep4) | (__builtin_amdgcn_alignbit(y, y, rot4) & ~keep4);
        y = uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x4e, 0xf, 0xf, true));
        x = (x & keep2) | (__builtin_amdgcn_alignbit(y, y, rot2) & ~keep2);
        y = uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xb1, 0xf, 0xf, true));
        v[i] = (x & keep1) | (__builtin_amdgcn_alignbit(y, y, rot1) & ~keep1);
    }
    return (unsigned long long)v[0] | ((unsigned long long)v[1] << 32);
}

// Superblock and entries [lo, hi) of chunk c; first chunk of the superblock in `first`
struct SbChunk {
    int sb;
    uint32_t lo, hi, first;
};
template <uint32_t kSbChunk>
__device__ inline SbChunk sb_chunk(const SbTable *T, uint32_t c) {
    // last superblock whose first chunk is <= c, 64 and then 16 candidates at a time
    const int lane = threadIdx.x & 63;
    constexpr int kFan = kMaxSb / 64;
    static_assert(kFan <= 64, "one candidate per lane");
    const auto count = [](bool v) { return __popcll(__builtin_amdgcn_ballot_w64(v)); };
    const int p = count(T->chunk[lane * kFan] <= c) - 1;
    const int a = p * kFan + count(lane < kFan && T->chunk[p * kFan + lane % kFan] <= c) - 1;
    SbChunk C;
    C.sb = a;
    C.first = T->chunk[a];
    C.lo = T->start[a] + (c - C.first) * kSbChunk;
    C.hi = C.lo + kSbChunk < T->start[a + 1] ? C.lo + kSbChunk : T->start[a + 1];
    return C;
}
// Tile of bit `bit` of superblock sb, or -1 outside the grid
__device__ inline int32_t sb_tile(const SbGrid &G, int sb, int bit) {
    const int32_t tx = (sb % G.sx) * kSbEdge + (bit & (kSbEdge - 1));
    const int32_t ty = (sb / G.sx) * kSbEdge + (bit >> kSbShift);
    return tx < G.gx && ty < G.gy ? ty * G.gx + tx : -1;
}

// Per chunk and tile of its superblock the number of entries that cover it (counts[chunk][tile]),
// added up per tile in ranges[tile].y. Integer sums: the order of the atomics does not matter.
template <int kSbChunk>
__global__ __launch_bounds__(256) void k_sb_count(const unsigned long long *e_mask,
                                                  const SbTable *T, SbGrid G, uint16_t *counts,
                                                  uint32_t *ranges) {
    constexpr int kSbGroups = kSbChunk / 64;
    __shared__ uint32_t s_c[4][kSbTiles];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint32_t n_chunks = T->chunk[kMaxSb];
    for (uint32_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const SbChunk C = sb_chunk<kSbChunk>(T, c);
        uint32_t cnt = 0;
#pragma unroll
        for (int g = 0; g < kSbGroups / 4; ++g) {
            const uint32_t e = C.lo + (g * 4 + w) * 64 + lane;
            const unsigned long long m = e < C.hi ? e_mask[e] : 0ull;
            cnt += uint32_t(__popcll(transpose64(m, lane)));
        }
        s_c[w][lane] = cnt;
        __syncthreads();
        if (t < kSbTiles) {
            const uint32_t sum = s_c[0][t] + s_c[1][t] + s_c[2][t] + s_c[3][t];
            counts[int64_t(c) * kSbTiles + t] = uint16_t(sum);
            const int32_t tile = sb_tile(G, C.sb, t);
            if (sum != 0u && tile >= 0) atomicAdd(&ranges[2 * int64_t(tile) + 1], sum);
        }
        __syncthreads();
    }
}

// Place of the sum before group j >= 1 of the superblock whose first chunk is `first`: a superblock's
// places start behind those of the one before, as its chunks do.
__device__ inline int64_t sb_group_place(uint32_t first, uint32_t j) { return int64_t(first / kSbGroup + j); }

// A superblock of more than kSbGroup chunks: per group j >= 1 and tile the pairs in the groups before
// it. Two steps: the groups' own sums, a wavefront each, then their running sum.
__device__ inline void sb_group_sums(const uint16_t *counts, uint32_t first, uint32_t chunks, uint32_t *groups) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t last = (chunks - 1) / kSbGroup;           // the last group
    for (uint32_t j = w; j < last; j += kScanTopThreads / 64) {
        const uint16_t *c = counts + (int64_t(first) + int64_t(j) * kSbGroup) * kSbTiles + lane;
        uint32_t sum = 0;
#pragma unroll 16
        for (int k = 0; k < kSbGroup; ++k) sum += c[k * kSbTiles];
        groups[sb_group_place(first, j + 1) * kSbTiles + lane] = sum;
    }
    __syncthreads();
    if (w != 0) return;
    uint32_t run = 0;
    for (uint32_t j = 1; j <= last; j += 8) {
        uint32_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            v[k] = groups[sb_group_place(first, j + k <= last ? j + k : last) * kSbTiles + lane];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            run += v[k];
            if (j + k <= last) groups[sb_group_place(first, j + k) * kSbTiles + lane] = run;
        }
    }
}

// Block 0: ranges[tile].y holds the list length: [start, end) in tile order, [0, 0) for an empty list.
// One block (at most 65536 tiles) that takes 16384 tiles at a time, moved through LDS so that memory is
// read and written in order (each thread reading its own 16 tiles took 35 us at 4K, now 13). Also
// the header's pair count and the capacity status.
// The other blocks, kSumBlocks where there are superblocks to look at: the sums of the superblocks b - 1,
// b - 1 + kSumBlocks, ... with many chunks (few or none: while block 0 scans, on compute units of their own).
constexpr int kSumBlocks = 64;
__global__ __launch_bounds__(kScanTopThreads) void k_tile_scan(uint2 *ranges, int32_t n_tiles,
                                                               BinHeader *hdr, int64_t cap,
                                                               int32_t *status, const SbTable *T,
                                                               const uint16_t *counts, uint32_t *groups) {
    if (blockIdx.x > 0) {                                    // block-uniform
        static_assert(kMaxSb <= 64 * kSumBlocks, "a lane for each superblock");
        const int sb0 = int(blockIdx.x) - 1 + int(threadIdx.x & 63) * kSumBlocks;
        uint32_t first = 0, chunks = 0;
        if (sb0 < kMaxSb) {
            first = T->chunk[sb0];
            chunks = T->chunk[sb0 + 1] - first;
        }
        unsigned long long many = __ballot(chunks > uint32_t(kSbGroup));
        while (many) {                                       // (the same in every wavefront)
            const int src = __ffsll((long long)many) - 1;
            many &= many - 1;
            sb_group_sums(counts, uint32_t(__builtin_amdgcn_readlane(int(first), src)),
                          uint32_t(__builtin_amdgcn_readlane(int(chunks), src)), groups);
        }
        return;
    }
    constexpr int kItems = 16, kStep = kScanTopThreads * kItems;
    __shared__ uint32_t s_v[kStep + kStep / kItems];         // a word of padding per thread's items
    __shared__ uint32_t s_wave[kScanTopThreads / 64];
    const int t = threadIdx.x;
    const auto at = [](int i) { return i + i / kItems; };
    uint32_t carry = 0;
    for (int32_t base = 0; base < n_tiles; base += kStep) {
        uint32_t v[kItems], sum = 0, tot;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int32_t i = base + k * kScanTopThreads + t;
            v[k] = i < n_tiles ? ranges[i].y : 0u;
        }
#pragma unroll
        for (int k = 0; k < kItems; ++k) s_v[at(k * kScanTopThreads + t)] = v[k];
        __syncthreads();
        uint32_t own[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            own[k] = s_v[at(t * kItems + k)];
            sum += own[k];
        }
        uint32_t run = block_exclusive_scan<uint32_t>(sum, s_wave, tot) + carry;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            s_v[at(t * kItems + k)] = run;
            run += own[k];
        }
        carry += tot;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int32_t i = base + k * kScanTopThreads + t;
            const uint32_t first = s_v[at(k * kScanTopThreads + t)];
            if (i < n_tiles && v[k] != 0u) ranges[i] = make_uint2(first, first + v[k]);
        }
        __syncthreads();
    }
    if (t == 0) {
        const unsigned long long total = hdr->total, ucap = (unsigned long long)cap;
        hdr->pairs = total < ucap ? total : ucap;
        if (total > ucap) *status = GSB_ERR_CAPACITY;
    }
}

// The lists. Lane t of a wavefront owns tile t: from the chunk's counts it knows where its part of
// the tile's list starts in LDS and steps through the set bits of its transposed masks, writing the
// entries' and the tile's numbers there; the block then copies the runs out, one element per thread
// and step, as the entries' Gaussian indices (looked up there, where every lane has one, not in the
// uneven steps before, and not tile by tile, where each step waits for the last: 109 us at 4K, now
// 79). A chunk's pairs go
// through LDS at once when they fit kSbStage, else in halves, quarters or two groups of 64 entries
// (at most kSbStage pairs) at a time. (Six wavefronts per SIMD: left alone, a few registers more make it
// five and the lists of 1 M Gaussians at 1080p 27 us, not 21.7.)
template <int kSbChunk>
__global__ __launch_bounds__(256, 6) void k_sb_write(const uint32_t *e_idx,
                                                  const unsigned long long *e_mask,
                                                  const SbTable *T, SbGrid G,
                                                  const uint16_t *counts, const uint32_t *groups,
                                                  const uint2 *ranges, uint32_t *point_list) {
    constexpr int kSbGroups = kSbChunk / 64;
    __shared__ uint32_t s_idx[kSbChunk];
    __shared__ uint16_t s_cnt[kSbGroups][kSbTiles];
    __shared__ uint32_t s_pre[4][kSbTiles];
    __shared__ uint16_t s_out[kSbStage];                     // tile * kSbChunk + entry of the chunk
    __shared__ uint32_t s_dst[kSbTiles];                     // list position of s_out[0] as a tile's
    static_assert(kSbTiles * kSbChunk <= 65536, "a tile and an entry fit 16 bits");
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint32_t n_chunks = T->chunk[kMaxSb];
    for (uint32_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const SbChunk C = sb_chunk<kSbChunk>(T, c);
        unsigned long long hit[kSbGroups / 4];
#pragma unroll
        for (int g = 0; g < kSbGroups / 4; ++g) {
            const int gr = g * 4 + w;
            const uint32_t e = C.lo + gr * 64 + lane;
            s_idx[gr * 64 + lane] = e < C.hi ? e_idx[e] : 0u;
            hit[g] = transpose64(e < C.hi ? e_mask[e] : 0ull, lane);
            s_cnt[gr][lane] = uint16_t(__popcll(hit[g]));
        }
        // the tile's entries in the superblock's earlier chunks: the groups before the chunk's own, and
        // the chunks of that. (All earlier chunks one by one: 3 M Gaussians on 128 x 128 px, 2930
        // chunks, took 193 us, now 59; 10 M 1581, now 152.)
        const uint32_t group = (c - C.first) / kSbGroup;
        uint32_t before = 0;
        if (w == 0 && group > 0)
            before = groups[sb_group_place(C.first, group) * kSbTiles + lane];
#pragma unroll 1
        for (uint32_t r = C.first + group * kSbGroup + w; r < c; r += 4)
            before += counts[int64_t(r) * kSbTiles + lane];
        s_pre[w][lane] = before;
        __syncthreads();
        const int32_t tile = sb_tile(G, C.sb, lane);
        uint32_t dst = s_pre[0][lane] + s_pre[1][lane] + s_pre[2][lane] + s_pre[3][lane] +
                       (tile >= 0 ? ranges[tile].x : 0u);    // the chunk's first pair of the tile
        // pairs of each quarter of the chunk (at most 2^14, two to a word), then how many groups of
        // 64 entries go through LDS at a time
        uint32_t q01 = 0, q23 = 0;
#pragma unroll
        for (int g = 0; g < kSbGroups / 4; ++g) {
            q01 += s_cnt[g][lane] | (uint32_t(s_cnt[kSbGroups / 4 + g][lane]) << 16);
            q23 += s_cnt[kSbGroups / 2 + g][lane] |
                   (uint32_t(s_cnt[3 * kSbGroups / 4 + g][lane]) << 16);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            q01 += __shfl_xor(q01, o, 64);
            q23 += __shfl_xor(q23, o, 64);
        }
        q01 = __builtin_amdgcn_readfirstlane(q01);
        q23 = __builtin_amdgcn_readfirstlane(q23);
        const uint32_t q[4] = {q01 & 0xffffu, q01 >> 16, q23 & 0xffffu, q23 >> 16};
        const auto fits = [](uint32_t pairs) { return pairs <= uint32_t(kSbStage); };
        const int ng = fits(q[0] + q[1] + q[2] + q[3]) ? kSbGroups
                     : fits(q[0] + q[1]) && fits(q[2] + q[3]) ? kSbGroups / 2
                     : fits(q[0]) && fits(q[1]) && fits(q[2]) && fits(q[3]) ? kSbGroups / 4 : 2;
        for (int g0 = 0; g0 < kSbGroups; g0 += ng) {         // block-uniform
            uint32_t len = 0;
            for (int g = g0; g < g0 + ng; ++g) len += s_cnt[g][lane];
            uint32_t x = len;                                // exclusive scan over the tiles
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            const uint32_t first = x - len;
            if (w == 0) s_dst[lane] = dst - first;
            uint32_t p = first;
            int seen = g0;                                   // groups whose counts p includes
#pragma unroll
            for (int k = 0; k < kSbGroups / 4; ++k) {
                const int g = k * 4 + w;
                if (g < g0 || g >= g0 + ng) continue;        // uniform
                for (; seen < g; ++seen) p += s_cnt[seen][lane];
                uint32_t o = p, lo = uint32_t(hit[k]), hi = uint32_t(hit[k] >> 32);
                uint32_t e = uint32_t(lane * kSbChunk + g * 64);
                while ((lo | hi) != 0u) {
                    if (lo == 0u) { lo = hi; hi = 0u; e += 32; }
                    s_out[o++] = uint16_t(e + __builtin_ctz(lo));
                    lo &= lo - 1u;
                }
            }
            __syncthreads();
            const uint32_t n_out = __builtin_amdgcn_readlane(x, 63);
#pragma unroll 4
            for (uint32_t j = t; j < n_out; j += 256) {
                const uint32_t v = s_out[j];
                point_list[s_dst[v / kSbChunk] + j] = s_idx[v % kSbChunk];
            }
            dst += len;
            __syncthreads();
        }
    }
}

// Few Gaussians on a small grid (n <= kSmallSort, few_lists): steps 1 to 4 in one launch, a block per
// superblock. Every block counts all tiles, from the rectangles' corners in a table of differences, and
// so knows where its own tiles' lists start; wave w then owns `per` chunks of 64 ranks, whose masks it
// transposes, and its lanes, a tile each, write the set bits' Gaussians. 2000 Gaussians on 16 tiles:
// 14 us and one launch, against 29 us in four.
constexpr int kListThreads = 1024, kListEdge = 128, kListCells = 9216;
constexpr int kListPer = kSmallSort / kListThreads;
inline bool few_lists(const SbGrid &G) {
    return G.gx <= kListEdge && G.gy <= kListEdge && (G.gx + 1) * (G.gy + 1) <= kListCells;
}
__global__ __launch_bounds__(kListThreads) void k_few_lists(const unsigned long long *rank_rects,
                                                            const uint32_t *sorted_idx, int n, SbGrid G,
                                                            BinHeader *hdr, int64_t cap, uint2 *ranges,
                                                            uint32_t *point_list, int32_t *status) {
    constexpr int kWaves = kListThreads / 64;
    __shared__ uint32_t s_cell[kListCells];        // differences, counts, then starts, stride gx + 1
    __shared__ uint32_t s_idx[kSmallSort];
    __shared__ uint32_t s_cnt[kWaves][kSbTiles];
    __shared__ uint32_t s_wave[kWaves];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int stride = G.gx + 1, cells = stride * (G.gy + 1), n_tiles = G.gx * G.gy;
    const unsigned long long all = hdr->total;
    if (all > (unsigned long long)cap) {                     // block-uniform: every list stays empty
        if (blockIdx.x == 0 && t == 0) {
            hdr->pairs = (unsigned long long)cap;
            *status = GSB_ERR_CAPACITY;
        }
        return;
    }
    if (blockIdx.x == 0 && t == 0) hdr->pairs = all;
    for (int i = t; i < cells; i += kListThreads) s_cell[i] = 0u;
    __syncthreads();
    const int per = ((n + 63) / 64 + kWaves - 1) / kWaves;   // <= kListPer
    unsigned long long rect[kListPer];
#pragma unroll
    for (int k = 0; k < kListPer; ++k) {
        const int j = (w * per + k) * 64 + lane;
        const bool valid = k < per && j < n;
        rect[k] = valid ? rank_rects[j] : 0ull;
        if (valid) s_idx[j] = sorted_idx[j];
    }
#pragma unroll
    for (int k = 0; k < kListPer; ++k) {
        const Rect R = unpack_rect(rect[k]);
        if (R.tx1 <= R.tx0 || R.ty1 <= R.ty0) continue;
        atomicAdd(&s_cell[R.ty0 * stride + R.tx0], 1u);
        atomicAdd(&s_cell[R.ty0 * stride + R.tx1], ~0u);
        atomicAdd(&s_cell[R.ty1 * stride + R.tx0], ~0u);
        atomicAdd(&s_cell[R.ty1 * stride + R.tx1], 1u);
    }
    __syncthreads();
    for (int y = w; y < G.gy; y += kWaves) {                 // sums along the rows
        uint32_t carry = 0;
        for (int x0 = 0; x0 < G.gx; x0 += 64) {
            const int x = x0 + lane;
            uint32_t v = x < G.gx ? s_cell[y * stride + x] : 0u;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(v, o, 64);
                if (lane >= o) v += u;
            }
            v += carry;
            if (x < G.gx) s_cell[y * stride + x] = v;
            carry = __shfl(v, 63, 64);
        }
    }
    __syncthreads();
    if (t < G.gx) {                                          // and along the columns
        uint32_t v = 0;
        for (int y = 0; y < G.gy; ++y) s_cell[y * stride + t] = v += s_cell[y * stride + t];
    }
    __syncthreads();
    constexpr int kOwn = kListCells / kListThreads;          // the tiles' starts
    uint32_t c[kOwn], sum = 0, tot;
    const int own = (n_tiles + kListThreads - 1) / kListThreads, i0 = t * own;
    int y = i0 / G.gx, x = i0 % G.gx;
    const int y0 = y, x0 = x;
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
        c[k] = 0u;
        if (k < own && i0 + k < n_tiles) {
            sum += c[k] = s_cell[y * stride + x];
            if (++x == G.gx) {
                x = 0;
                ++y;
            }
        }
    }
    uint32_t run = block_exclusive_scan<uint32_t>(sum, s_wave, tot);
    y = y0;
    x = x0;
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
        if (k < own && i0 + k < n_tiles) {
            s_cell[y * stride + x] = run;
            run += c[k];
            if (++x == G.gx) {
                x = 0;
                ++y;
            }
        }
    }
    const int sx = int(blockIdx.x) % G.sx, sy = int(blockIdx.x) / G.sx;
    unsigned long long hit[kListPer];
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 0; k < kListPer; ++k) {
        const Rect R = unpack_rect(rect[k]);
        unsigned long long m = 0;
        if (R.tx0 < (sx + 1) * kSbEdge && R.tx1 > sx * kSbEdge && R.ty0 < (sy + 1) * kSbEdge &&
            R.ty1 > sy * kSbEdge && R.tx0 < R.tx1 && R.ty0 < R.ty1)
            m = sb_mask(sb_span(R.tx0, R.tx1, sx) | (sb_span(R.ty0, R.ty1, sy) << 8));
        hit[k] = transpose64(m, lane);
        cnt += uint32_t(__popcll(hit[k]));
    }
    s_cnt[w][lane] = cnt;
    __syncthreads();
    const int tx = sx * kSbEdge + (lane & (kSbEdge - 1)), ty = sy * kSbEdge + (lane >> kSbShift);
    if (tx >= G.gx || ty >= G.gy) return;                    // (no barrier below)
    uint32_t o = s_cell[ty * stride + tx], len = 0;
    const uint32_t first = o;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const uint32_t e = s_cnt[k][lane];
        o += k < w ? e : 0u;
        len += e;
    }
    if (w == 0 && len > 0) ranges[ty * G.gx + tx] = make_uint2(first, first + len);
#pragma unroll
    for (int k = 0; k < kListPer; ++k) {
        const uint32_t *idx = s_idx + (w * per + k) * 64;
        for (unsigned long long m = hit[k]; m != 0ull; m &= m - 1ull)
            if (o < cap) point_list[o++] = idx[__ffsll((long long)m) - 1];
    }
}

// Start of bin_fill: empty ranges, zeroed sort states, the Gaussian count for the depth sort and
// a clean status word (later kernels only ever write error codes into it).
__global__ __launch_bounds__(256) void k_bin_init(uint32_t *ranges, int64_t m, SortState *sorts,
                                                  BinHeader *hdr, int64_t n, SbTable *table,
                                                  int32_t *status) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < m) ranges[i] = 0u;
    if (blockIdx.x == 0) {
        uint32_t *w = reinterpret_cast<uint32_t *>(sorts);
        for (int k = threadIdx.x; k < int(sizeof(SortState) / 4); k += blockDim.x) w[k] = 0u;
        if (table && threadIdx.x < kSbLists) table->listed[threadIdx.x][0] = 0ull;
        if (threadIdx.x == 0) {
            hdr->gaussians = (unsigned long long)n;
            *status = GSB_OK;
        }
    }
}

// Tile boundaries in the sorted tile ids: four consecutive pairs per thread (one vector load and
// the two neighbours outside it). `tiles` is 256-byte aligned.
template <typename K>
__global__ __launch_bounds__(256) void k_ranges(const K *tiles, const unsigned long long *count,
                                                uint32_t *ranges) {
    const int64_t P = int64_t(*count);
    const int64_t i0 = 4 * (int64_t(blockIdx.x) * blockDim.x + threadIdx.x);
    if (i0 >= P) return;
    uint32_t t[6];                       // tiles[i0 - 1 .. i0 + 4]; outside [0, P): no tile
    t[0] = i0 > 0 ? tiles[i0 - 1] : 0xffffffffu;
    if (i0 + 4 <= P) {
        const uint4 v = load4(tiles, i0);
        t[1] = v.x; t[2] = v.y; t[3] = v.z; t[4] = v.w;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) t[1 + k] = i0 + k < P ? tiles[i0 + k] : 0xffffffffu;
    }
    t[5] = i0 + 4 < P ? tiles[i0 + 4] : 0xffffffffu;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t i = i0 + k;
        if (i >= P) break;
        if (t[k] != t[k + 1]) ranges[2 * int64_t(t[k + 1])] = uint32_t(i);
        if (t[k + 2] != t[k + 1]) ranges[2 * int64_t(t[k + 1]) + 1] = uint32_t(i + 1);
    }
}

int ceil_log2(int64_t v) {
    int b = 0;
    while ((int64_t(1) << b) < v) ++b;
    return b;
}

}  // namespace

size_t bin_workspace_bytes(int64_t n, int64_t pair_capacity, int64_t /*n_tiles*/) {
    // bin_count uses the leading part, which does not depend on the capacity; bin_fill all of it
    return layout(n, pair_capacity).end;
}

int64_t bin_max_gaussians() { return kScanMaxLen; }
// the tile sort scans [256][blocks] histograms with the single-top-level scan
int64_t bin_max_pairs() { return int64_t(kScanMaxLen / kRadix) * kSortTile; }

gsb_status bin_count(const float *means2d, const int32_t *radii, const float *conics,
                     const float *opacity, int32_t mode, int64_t n, int32_t W, int32_t H, void *ws,
                     int64_t *n_pairs_dev, hipStream_t s) {
    const Layout L = layout(n, 0);
    auto *hdr = at<BinHeader>(ws, L.hdr);
    auto *counts = at<unsigned long long>(ws, L.counts);
    auto *masks = at<unsigned long long>(ws, L.masks);
    auto *recs = at<uint4>(ws, L.recs);
    auto *partial = at<unsigned long long>(ws, L.partials);
    auto *total_b = reinterpret_cast<long long *>(n_pairs_dev);
    const auto *means = reinterpret_cast<const float2 *>(means2d);
    const int32_t gx = int32_t(grid_x(W)), gy = int32_t(grid_y(H));
    // Gaussians per block: mode 0 one block up to 4096 (no second launch), then 1024; mode 1, whose
    // tests are long, 256; more where the blocks would exceed the partial sums' place
    if (by_superblock(sb_grid(gx, gy))) counts = nullptr;
    int64_t nb = 0;
    const auto blocks = [&](int per) { return dim3(unsigned(nb = (n + per - 1) / per)); };
    constexpr int64_t kTop = kScanMaxBlocks;
    if (n > 0 && mode == GSB_BIN_RECT && n <= 4096) {
        k_bin_count<0, 1024><<<blocks(4096), 1024, 0, s>>>(means, radii, conics, opacity, n, 4, gx, gy,
                                                           W, H, counts, masks, recs, partial,
                                                           &hdr->total, total_b);
    } else if (n > 0 && mode == GSB_BIN_RECT) {
        const int iters = n <= 1024 * kTop ? 4 : 16;
        k_bin_count<0, 256><<<blocks(256 * iters), 256, 0, s>>>(means, radii, conics, opacity, n,
                                                                iters, gx, gy, W, H, counts, masks,
                                                                recs, partial, &hdr->total, total_b);
    } else if (n > 0) {
        const int iters = n <= 256 * kTop ? 1 : n <= 1024 * kTop ? 4 : 16;
        k_bin_count<1, 256><<<blocks(256 * iters), 256, 0, s>>>(means, radii, conics, opacity, n,
                                                                iters, gx, gy, W, H, counts, masks,
                                                                recs, partial, &hdr->total, total_b);
    }
    // the total only: offsets are formed in depth order by bin_fill
    if (nb != 1)
        k_scan_top<unsigned long long><<<1, kScanTopThreads, 0, s>>>(partial, nb, &hdr->total, total_b);
    return check_launch("bin_count");
}

// bin_fill's part that needs no capacity: empty ranges, clean states and status word, and the
// Gaussians in depth order (ties by index: the sort is stable over index order). The last pass also
// lays out in rank order each Gaussian's rectangle and its pair count or mask.
gsb_status bin_sort(int32_t mode, const float *depths, int64_t n, int32_t W, int32_t H, void *ws,
                    uint32_t *ranges, int32_t *status_dev, hipStream_t s) {
    const Layout L = layout(n, 0);       // (the look-back words' place in the smallest workspace)
    auto *hdr = at<BinHeader>(ws, L.hdr);
    auto *sorts = at<SortState>(ws, L.sorts);
    uint32_t *dka = at<uint32_t>(ws, L.dkey_a), *dkb = at<uint32_t>(ws, L.dkey_b);
    uint32_t *dva = at<uint32_t>(ws, L.dval_a), *dvb = at<uint32_t>(ws, L.dval_b);
    const int64_t n_tiles = grid_x(W) * grid_y(H);
    const bool sb = by_superblock(sb_grid(int32_t(grid_x(W)), int32_t(grid_y(H))));
    auto *rank_counts = sb && mode == GSB_BIN_RECT ? nullptr : at<unsigned long long>(ws, L.offs);
    auto *rects = at<unsigned long long>(ws, L.rects);
    if (sb && n > 0 && n <= kRankSort) {
        const size_t lds = sizeof(uint32_t) * size_t((n + 63) & ~int64_t(63));
        k_rank<<<dim3(unsigned((n + 63) / 64)), kRankThreads, lds, s>>>(
            depths, int(n), dva, at<uint4>(ws, L.recs), rank_counts, rects, ranges, int(2 * n_tiles),
            at<SbTable>(ws, L.sb_table), status_dev);
        return check_launch("bin_sort");
    }
    k_bin_init<<<dim3(unsigned((2 * n_tiles + 255) / 256)), 256, 0, s>>>(
        ranges, 2 * n_tiles, sorts, hdr, n, at<SbTable>(ws, L.sb_table), status_dev);
    // the look-back words of the smaller tiles (4096 bytes per 1024 Gaussians) take the place of the
    // masks by index (8 bytes per Gaussian, and n > kRankSort here), which superblocks do not use
    if (sb && n > 0 && n <= kSort4)
        sort_depth<4>(depths, dka, dkb, dva, dvb, &hdr->gaussians, n, sorts, at<uint32_t>(ws, L.masks),
                      status_dev, at<uint4>(ws, L.recs), rank_counts, rects, s);
    else if (n > 0)
        sort_depth<kSortItems>(depths, dka, dkb, dva, dvb, &hdr->gaussians, n, sorts,
                               at<uint32_t>(ws, L.sortbuf), status_dev, at<uint4>(ws, L.recs),
                               rank_counts, rects, s);
    return check_launch("bin_sort");
}

gsb_status bin_fill_sorted(const float *means2d, const float *conics, const float *opacity,
                           int32_t mode, int64_t n, int32_t W, int32_t H, void *ws,
                           uint32_t *point_list, int64_t cap, uint32_t *ranges,
                           int32_t *status_dev, hipStream_t s) {
    const Layout L = layout(n, cap);
    auto *hdr = at<BinHeader>(ws, L.hdr);
    auto *counts = at<unsigned long long>(ws, L.counts);
    auto *partial64 = at<unsigned long long>(ws, L.partials);
    auto *partial32 = at<uint32_t>(ws, L.partials);
    auto *sortbuf = at<uint32_t>(ws, L.sortbuf);
    uint32_t *dka = at<uint32_t>(ws, L.dkey_a), *dkb = at<uint32_t>(ws, L.dkey_b);
    const uint32_t *dva = at<uint32_t>(ws, L.dval_a);
    auto *offs = at<unsigned long long>(ws, L.offs);
    uint32_t *vtmp = at<uint32_t>(ws, L.vals_tmp);
    const int32_t gx = int32_t(grid_x(W)), gy = int32_t(grid_y(H));
    const int64_t n_tiles = int64_t(gx) * gy;
    const unsigned gn = unsigned(n > 0 ? (n + 255) / 256 : 1);

    const SbGrid G = sb_grid(gx, gy);
    if (by_superblock(G) && n > 0 && cap > 0) {
        const auto *rects = at<unsigned long long>(ws, L.rects);
        auto *e_mask = at<unsigned long long>(ws, L.sb_mask);
        auto *e_idx = at<uint32_t>(ws, L.sb_idx);
        auto *counts16 = at<uint16_t>(ws, L.sb_counts);
        auto *groups = at<uint32_t>(ws, L.sb_groups);
        auto *table = at<SbTable>(ws, L.sb_table);
        const int bits = G.n > 1 ? ceil_log2(G.n) : 0;
        const int chunk = sb_chunk_size(cap);
        // mode 1: the masks in rank order (in the offsets' place), the large rectangles' masks from
        // the end of the entries' masks downwards
        const bool vis = mode == GSB_BIN_VISIBLE;
        auto *rank_masks = vis ? offs : nullptr;
        const SbVisible V{rank_masks, at<uint4>(ws, L.recs), e_mask + cap, e_idx + cap, table, n > 1 << 16 ? kSbLists : 1,
                          reinterpret_cast<const float2 *>(means2d), conics, opacity, W, H};
        if (vis)
            k_sb_list<<<dim3(unsigned((n + 63) / 64)), 64, 0, s>>>(V, table, n, G, cap);
        if (n <= kSmallSort && !vis && few_lists(G)) {
            k_few_lists<<<dim3(unsigned(G.n)), kListThreads, 0, s>>>(
                rects, dva, int(n), G, hdr, cap, reinterpret_cast<uint2 *>(ranges), point_list, status_dev);
            return check_launch("bin_fill");
        }
        if (n <= kSmallSort && !vis && double(n) * sb_entries(n, cap) <= kSbOneEntries) {
            const auto scatter = n <= 4 * kSortThreads ? k_sb_scatter<4, true, false>
                               : n <= 8 * kSortThreads ? k_sb_scatter<8, true, false>
                                                       : k_sb_scatter<16, true, false>;
            const int ranks = kSortThreads * (n <= 4 * kSortThreads ? 4 : n <= 8 * kSortThreads ? 8 : 16);
            scatter<<<1, kSortThreads, 0, s>>>(rects, dva, n, ranks, G, bits, nullptr, 1, hdr, cap, chunk, e_idx,
                                               e_mask, table, V, nullptr, nullptr);
        } else {
            const int ranks = sb_ranks(G.n, n, cap);
            const int64_t nblk = (n + ranks - 1) / ranks;
            const dim3 gb{unsigned(xcd_grid(nblk))};
            if (vis)
                k_sb_hist_visible<<<gb, kSortThreads, 0, s>>>(rects, dva, V, n, ranks, G, sortbuf, nblk,
                                                              cap, dka, dkb);
            else
                k_sb_hist<<<gb, kSortThreads, 0, s>>>(rects, n, ranks, G, sortbuf, nblk);
            launch_scan<uint32_t>(sortbuf, int64_t(G.n) * nblk, partial32, &hdr->entries, nullptr, s);
            const auto scatter =
                ranks <= 256 ? (vis ? k_sb_scatter<1, false, true> : k_sb_scatter<1, false, false>)
              : ranks <= 1024 ? (vis ? k_sb_scatter<4, false, true> : k_sb_scatter<4, false, false>)
              : ranks == 2048 ? (vis ? k_sb_scatter<8, false, true> : k_sb_scatter<8, false, false>)
                              : (vis ? k_sb_scatter<16, false, true> : k_sb_scatter<16, false, false>);
            scatter<<<gb, kSortThreads, 0, s>>>(rects, dva, n, ranks, G, bits, sortbuf, nblk, hdr, cap, chunk,
                                                e_idx, e_mask, table, V, dka, dkb);
        }
        const int64_t mc = sb_max_chunks(cap);
        const dim3 gc{unsigned(mc < kSbMaxGrid ? mc : kSbMaxGrid)};
        const auto count = chunk == kSbChunkSmall ? k_sb_count<kSbChunkSmall> : k_sb_count<kSbChunkLarge>;
        const auto write = chunk == kSbChunkSmall ? k_sb_write<kSbChunkSmall> : k_sb_write<kSbChunkLarge>;
        count<<<gc, 256, 0, s>>>(e_mask, table, G, counts16, ranges);
        k_tile_scan<<<1 + kSumBlocks, kScanTopThreads, 0, s>>>(
            reinterpret_cast<uint2 *>(ranges), int32_t(n_tiles), hdr, cap, status_dev, table, counts16,
            groups);
        write<<<gc, 256, 0, s>>>(e_idx, e_mask, table, G, counts16, groups,
                                 reinterpret_cast<const uint2 *>(ranges), point_list);
        return check_launch("bin_fill");
    }
    if (by_superblock(G)) {       // no Gaussians, or no room for a pair
        k_tile_scan<<<1, kScanTopThreads, 0, s>>>(reinterpret_cast<uint2 *>(ranges), 0, hdr, cap,
                                                  status_dev, nullptr, nullptr, nullptr);
        return check_launch("bin_fill");
    }
    const uint32_t *sorted_idx = dva;
    // (1. the depth sort) 2. offsets in rank order; pairs emitted in rank order
    launch_scan<unsigned long long>(offs, n, partial64, nullptr, nullptr, s);
    const int tile_bits = ceil_log2(n_tiles) > 0 ? ceil_log2(n_tiles) : 1;
    const int tp = (tile_bits + kRadixBits - 1) / kRadixBits;
    // the last pass must land the values in point_list
    uint32_t *v_first = (tp % 2 == 0) ? point_list : vtmp;
    uint32_t *v_second = (tp % 2 == 0) ? vtmp : point_list;
    // 3. stable sort of the pairs on the tile id; 4. the tiles' ranges. The emission stages 6144
    //    pairs per block when 256 ranks are expected to emit more than 3584 (capacity per Gaussian)
    const bool large_stage = n > 0 && 256.0 * double(cap) > 3584.0 * double(n);
    const auto emit_sort_range = [&](auto *tka, auto *tkb) {
        using K = std::remove_pointer_t<decltype(tka)>;
        const auto fill = large_stage ? k_bin_fill<K, kFillStageLarge> : k_bin_fill<K, kFillStage>;
        fill<<<gn, 256, 0, s>>>(reinterpret_cast<const float2 *>(means2d), conics, opacity, mode, W,
                                H, sorted_idx, n, gx, gy, offs, counts,
                                at<unsigned long long>(ws, L.masks),
                                at<unsigned long long>(ws, L.rects), hdr, cap, tka, v_first,
                                status_dev);
        sort_tiles<K>(tka, tkb, v_first, v_second, &hdr->pairs, cap, tile_bits, sortbuf,
                      partial32, status_dev, s);
        const K *tiles_sorted = (tp % 2 == 0) ? tka : tkb;
        if (cap > 0)
            k_ranges<K><<<dim3(unsigned((cap + 1023) / 1024)), 256, 0, s>>>(tiles_sorted,
                                                                             &hdr->pairs, ranges);
    };
    if (n_tiles <= kMaxTiles16)
        emit_sort_range(at<uint16_t>(ws, L.tkey_a), at<uint16_t>(ws, L.tkey_b));
    else
        emit_sort_range(at<uint32_t>(ws, L.tkey_a), at<uint32_t>(ws, L.tkey_b));
    return check_launch("bin_fill");
}

gsb_status bin_fill(const float *means2d, const float *conics, const float *opacity, int32_t mode,
                    const float *depths, int64_t n, int32_t W, int32_t H, void *ws,
                    uint32_t *point_list, int64_t cap, uint32_t *ranges,
                    int32_t *status_dev, hipStream_t s) {
    const gsb_status st = bin_sort(mode, depths, n, W, H, ws, ranges, status_dev, s);
    if (st != GSB_OK) return st;
    return bin_fill_sorted(means2d, conics, opacity, mode, n, W, H, ws, point_list, cap, ranges,
                           status_dev, s);
}

// ------------------------------------------------------------------------------- offsets
// The device scan for other steps that group by Gaussian (the deterministic backward); any length.
size_t offsets_scratch_bytes(int64_t n) {
    return sizeof(uint32_t) * size_t((n + kScanTile - 1) / kScanTile + 1);
}

void counts_to_offsets(const uint32_t *counts, uint32_t *offsets, int64_t n, void *scratch,
                       hipStream_t s) {
    auto *partial = static_cast<uint32_t *>(scratch);
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    const dim3 grid{unsigned(nb)};
    k_scan_reduce<uint32_t><<<grid, kScanThreads, 0, s>>>(counts, n, partial);
    k_scan_down_fused<uint32_t><<<grid, kScanThreads, 0, s>>>(counts, offsets, n, partial, nb, nullptr,
                                                             nullptr);
}

// ------------------------------------------------------------------------------- no-alloc binning
// Library-held binning workspace for callers that cannot allocate device memory. One copy of the
// array lives on every GPU the library runs on, at its own address, from module load to process
// end. In host code the name `scratch` only stands in for the symbol: its device address comes
// from hipGetSymbolAddress, once per device, with that device current, and only that address is
// passed to kernels.
static __device__ __align__(256) unsigned char scratch[GSB_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kScratchDevices];   // device address of `scratch` per device (null = not yet)
}  // namespace

gsb_status bin_noalloc(const float *means2d, const int32_t *radii, const float *conics,
                       const float *opacity, int32_t mode, const float *depths, int64_t n,
                       int32_t W, int32_t H, uint32_t *point_list, int64_t cap, uint32_t *ranges,
                       int64_t *n_pairs_dev, int32_t *status_dev, hipStream_t s) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(GSB_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kScratchDevices)
        return fail(GSB_ERR_UNSUPPORTED, "device id %d out of range", dev);
    void *ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (g_scratch_ptr[dev] == nullptr) {
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || p == nullptr)
                return fail(GSB_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
            g_scratch_ptr[dev] = p;
        }
        ws = g_scratch_ptr[dev];
    }
    // Every word of the workspace that the binning reads is written earlier in the same call
    // (counts, scans, the sort state and look-back words are initialised by its own kernels), so
    // what a previous call left in the array needs no clearing.
    const gsb_status st = bin_count(means2d, radii, conics, opacity, mode, n, W, H, ws,
                                    n_pairs_dev, s);
    if (st != GSB_OK) return st;
    return bin_fill(means2d, conics, opacity, mode, depths, n, W, H, ws, point_list, cap,
                    ranges, status_dev, s);
}

}  // namespace gsb
