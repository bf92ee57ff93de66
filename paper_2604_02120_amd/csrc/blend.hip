// Tile blending of depth-sorted projected 2D Gaussians on gfx950: forward (Eq. (volume-render)
// with the per-pixel loop of Alg. 1) and backward, with the Gaussian exponent evaluated either
//   PLAIN : per pixel on the vector ALUs in FP32 from Eq. (power), or
//   F16 / BF16 : as the product M_power = M_g . M_p of Eq. (power rewritten) / Eq. (matrix
//          multiplication) on the matrix cores (MFMA), FP16 or BF16 operands, FP32 accumulation.
//
// Launch shape: one 256-thread block (4 wavefronts) per 16x16 tile, one pixel per lane; wave w
// owns the 8x8 quadrant (w mod 2, w div 2) of the tile. The tile's sorted list is walked in
// batches of NB entries (a template parameter: 64, 128 or 256, 256 by default): every thread below
// NB fetches one (the next batch's global loads are issued before the current batch is composited)
// and, if the Gaussian can reach the tile (reaches_tile), stages it into the next free LDS slot;
// each wave composites the staged Gaussians for its pixels, 16 (one MFMA group) at a time.
// Of a 3-sigma list only 39% reach (4K frame of 3M Gaussians): staging all of them, 128 at a time,
// took 822 us forward and 2203 backward there (BF16), now 640 and 1976; lists that hold only
// reaching entries pay the test with nothing to drop (forward 541 -> 564 us, backward 2094 -> 1880
// with this and the column-first sums).
//
// Exponent in log2 units. With L = log2(e), every path evaluates
//     q = L * power + log2(o),   alpha = min(0.99, 2^min(q, log2 o))  (= min(0.99, o e^min(power,0)))
// and skips a pair when q < log2(1/255) (alpha < 1/255), so culled pairs never reach exp2. A
// Gaussian with o < 1/255 can never pass and is staged as inert.
//
// GEMM form. Relative to the tile centre (x_c, y_c) = (x0 + 7.5, y0 + 7.5) (the reference pixel of
// Eq. 4), pixel basis v_p = [xb^2, yb^2, xb yb, xb, yb] with xb = x_c - px (quarter-integers, exact
// in FP16 and BF16) and Gaussian row v_g = L [-A/2, -C/2, -B, -(A xh + B yh), -(C yh + B xh)] with
// xh = x - x_c; the constant term L(-A xh^2/2 - C yh^2/2 - B xh yh) + log2 o is the FP32
// accumulator init. v_g is split into hi + lo terms in the 16-bit format (lo scaled by 2^12 to stay
// clear of FP16 subnormals, with the basis scaled by 2^-12 for that product, both exact), so the two
// MFMAs recover ~22 (FP16) / ~16 (BF16) significant bits of v_g.
//
// Conditioning. Needle-like Gaussians (axis ratio up to ~100) make the quadratic form a sum of
// terms ~1e5 that cancel to O(1); evaluated naively in FP32 the exponent is off by up to ~1e-2.
// Both paths therefore evaluate Q = d^T Sigma^-1 d as dx*gx + dy*gy with g = Sigma^-1 d, where each
// product A*dx's rounding error is recovered exactly with an FMA and added back, so g (small along
// the needle, where the cancellation happens) carries full FP32 relative accuracy. The plain path
// does this per pair; the GEMM path once per staged Gaussian, for v_g[3], v_g[4] and the constant.
//
// MFMA packing (v_mfma_f32_32x32x16_{f16,bf16}): lane l supplies A[l%32][8(l/32)..+7] and
// B[8(l/32)..+7][l%32]; accumulator register v of lane l holds D[8(v/4) + 4(l/32) + v%4][l%32].
// B is each lane's own pixel basis. A is block-diagonal: row i carries v_g of Gaussian
// 4(i/8) + i%4 in k-block (i/4)%2 and zeros in the other, so register v of lane l ends up holding
// q of Gaussian v of the group for pixel l: one MFMA pair yields 16 Gaussians x 64 pixels in
// exactly the "lane = pixel, register = next Gaussian in depth order" layout that compositing
// needs, with no shuffles.
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>
#include <cstddef>
#include <type_traits>
#include <vector>

#include "gsb_internal.h"

namespace gsb {
namespace {

enum class Mode { Plain, F16, BF16 };

constexpr int kGroup = 16;                  // Gaussians per MFMA group
constexpr float kLog2e = 0x1.715476p+0f;    // log2(e) rounded to FP32
constexpr float kQCull = -0x1.ffa37cp+2f;   // log2(fp32(1/255)) rounded to FP32
constexpr float kTauCull = 1.0f / 255.0f;
constexpr float kAlphaMax = 0.99f;
// The 0.99 clamp applied before the exponential: v_exp_f32 is monotonic near log2(0.99) and
// returns exactly 0.99f for every input from -0x1.db1f6ep-7 to -0x1.db1eb8p-7 (checked over every
// FP32 input in [-0.03, -0.014]), so min(2^x, 0.99f) = 2^min(x, kQAlphaMax) bit for bit, one
// three-way min instead of two mins; 2^x >= 0.99f exactly when x >= kQAlphaMaxLo.
constexpr float kQAlphaMax = -0x1.db1f16p-7f;     // log2f(0.99f)
constexpr float kQAlphaMaxLo = -0x1.db1f6ep-7f;
constexpr float kTStop = 1e-4f;
constexpr float kLoScale = 4096.0f;         // 2^12
constexpr float kLoScaleInv = 1.0f / 4096.0f;
constexpr float kF16Max = 65504.0f;

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4x __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f16x __attribute__((ext_vector_type(16)));

template <Mode M> struct Op;
template <> struct Op<Mode::F16> {
    typedef h8 vec;
    static __device__ inline vec cvt(const float v[8]) {
        vec r;
#pragma unroll
        for (int k = 0; k < 8; ++k) r[k] = _Float16(fminf(fmaxf(v[k], -kF16Max), kF16Max));
        return r;
    }
    static __device__ inline float back(const vec &x, int k) { return float(x[k]); }
    static __device__ inline f16x mfma(vec a, vec b, f16x c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};
template <> struct Op<Mode::BF16> {
    typedef b8 vec;
    static __device__ inline vec cvt(const float v[8]) {
        vec r;
#pragma unroll
        for (int k = 0; k < 8; ++k) r[k] = __bf16(v[k]);
        return r;
    }
    static __device__ inline float back(const vec &x, int k) { return float(x[k]); }
    static __device__ inline f16x mfma(vec a, vec b, f16x c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Op<Mode::Plain> { typedef h8 vec; };

// ------------------------------------------------------------------------------- LDS staging
// Forward: one batch of the entries that can reach the tile, in list order.
template <Mode M, int NB>
struct FwdStage {              // GEMM form
    typedef typename Op<M>::vec vec;
    vec ahi[NB], zero, alo[NB];
    float kc[NB];
    float4 attr[NB];           // (log2 o, r, g, b)
    uint8_t pos[NB];           // the entry's place in the batch as fetched
    // per wavefront: entries it keeps, + kWaveLive while it has a live pixel
    alignas(16) uint32_t post[4];
};
template <int NB>
struct FwdStage<Mode::Plain, NB> {
    float4 geo[NB];            // (x, y, A, B)
    float2 geo2[NB];           // (C, log2 o)
    float4 attr[NB];
    uint8_t pos[NB];
    uint8_t reach[NB];         // reach_mask
    alignas(16) uint32_t post[4];
};
constexpr uint32_t kWaveLive = 1u << 16;

// Backward: the same, with what the reverse step needs besides.
template <int NB>
struct BwdSlots {
    float4 attr[NB];           // (log2 o, r, g, b)
    float2 mean[NB];
    // The Gaussian index of each slot (written after the barrier that ends the staging: the flush of
    // the batch before reads other threads' slots until then).
    uint32_t ids[NB];
    // which of its 64 entries each wavefront keeps
    alignas(16) unsigned long long kept[4];
};
template <Mode M, int NB>
struct BwdStage : BwdSlots<NB> {   // GEMM form
    typedef typename Op<M>::vec vec;
    vec ahi[NB];               // v_g hi terms, 5 used of 8
    vec zero_hi;               // zeros: the A operand of the lanes off the block diagonal
    vec alo[NB];               // v_g lo terms * 2^12
    vec zero_lo;               // zeros, as far from zero_hi as alo[i] is from ahi[i]
    float kc[NB];              // accumulator init: constant term + log2 o (-inf = inert)
};
template <int NB>
struct BwdStage<Mode::Plain, NB> : BwdSlots<NB> {
    float4 geo[NB];            // (x, y, A, B)
    float2 geo2[NB];           // (C, log2 o)
    uint8_t reach[NB];         // reach_mask
};

constexpr int kGrad = 9;   // per-Gaussian sums kept per batch
// Deterministic backward: the nine sums of a list position are one aligned 64-byte row.
constexpr int kDetStride = 16;

// dL/do from the sum of alpha dL/dalpha over the Gaussian's pairs (alpha = o e^power below the 0.99
// clamp): that sum over o. A Gaussian with o < 1/255 is never blended (its sum is zero).
__device__ inline float opacity_grad(float sum, float o) { return o >= kTauCull ? sum / o : 0.f; }

// Per-Gaussian gradient sums of a batch: 9 consecutive words per staged Gaussian, which the
// flush reads as consecutive words across lanes.
template <int NB>
struct BwdAcc {
    float v[NB * kGrad];
    // each wavefront's list of the slots with a nonzero sum, built when it flushes
    uint16_t list[kBlock / 64][64];
    // where lane l of a flush adds: the word l % 9 of its Gaussian, from `dst` at `stride` floats
    // per Gaussian (the same for the whole tile; kept here, not in three registers per lane)
    struct Item { float *dst; uint32_t stride, pad; } item[64];
};

// Deterministic backward: each wavefront adds its per-batch sums in a slice of its own (a fixed
// order); the flush adds the four slices in a fixed order. entry: the slots' places in the batch;
// list: each wavefront's slots with a nonzero sum.
constexpr int kNoSlot = 0xffff;
template <int NB>
struct BwdAccDet {
    float v[kBlock / 64][NB * kGrad];
    uint16_t entry[NB];
    uint16_t list[kBlock / 64][NB / (kBlock / 64)];
};

// Backward reduction on the matrix cores: each wavefront's dL/dpower values of 8 Gaussians for its
// 64 pixels (one word per (Gaussian, pixel): FP16 hi in the low half, FP16 lo x 2^12 in the high
// half), transposed through LDS into the operand of v_mfma_f32_16x16x32_f16. Rows padded to 68
// words. Row 0 doubles as the 8 x 8 table of the product's results (moments) once the operand has
// been read. The rows are zero whenever a half-group starts.
constexpr int kDgStride = 68;
struct alignas(16) BwdMM {
    uint32_t dg[kBlock / 64][8][kDgStride];
};

// Raw attributes of one list entry, fetched in the prefetch step.
struct GRaw {
    float x, y, A, B, C, o, r, g, b;
    uint32_t id;
    bool valid;
};

struct __attribute__((aligned(4))) F3 { float a, b, c; };

// a*x + b*y to full FP32 relative accuracy: the rounding error of a*x is recovered with an FMA.
__device__ inline float dot2_acc(float a, float x, float b, float y) {
    const float p = __fmul_rn(a, x);
    const float pe = fmaf(a, x, -p);
    return fmaf(b, y, p) + pe;
}
// Q = A dx^2 + 2 B dx dy + C dy^2 as dx*gx + dy*gy with g = Sigma^-1 (dx, dy) from dot2_acc.
__device__ inline float quad_acc(float A, float B, float C, float dx, float dy, float &gx, float &gy) {
    gx = dot2_acc(A, dx, B, dy);
    gy = dot2_acc(C, dy, B, dx);
    return fmaf(dx, gx, __fmul_rn(dy, gy));
}

// A list entry (Gaussian index) loaded ahead of its use. The load is unconditional (an invalid
// slot reads the list's entry `fallback`, which exists) and validity is applied only at the use,
// so that nothing waits for the load before then.
constexpr uint32_t kNoEntry = 0xffffffffu;
struct Entry {
    uint32_t raw;
    bool valid;
    __device__ uint32_t id() const { return valid ? raw : kNoEntry; }
};
__device__ inline Entry load_entry(const uint32_t *plist, int64_t pos, bool valid, int64_t fallback) {
    return Entry{plist[valid ? pos : fallback], valid};
}

// Attributes of the Gaussian `id` (from load_entry). Needs n > 0. An index >= n (kNoEntry, or an
// inconsistent list) gives an invalid entry, which stage() makes inert; its loads read Gaussian 0
// instead, so that no load is conditional: the loads of a batch stay in flight until the batch
// is staged, with no copies of their results (and no waits for them) in between.
__device__ inline GRaw fetch_attrs(uint32_t id, uint32_t n, const float2 *means, const F3 *conics,
                                   const float *opac, const F3 *colors) {
    GRaw g;
    g.valid = id < n;
    g.id = g.valid ? id : 0u;
    const float2 m = means[g.id];
    const F3 c = conics[g.id];
    const F3 col = colors[g.id];
    g.x = m.x; g.y = m.y; g.A = c.a; g.B = c.b; g.C = c.c;
    g.o = opac[g.id];
    g.r = col.a; g.g = col.b; g.b = col.c;
    return g;
}

// Where a tile's Gaussian attributes come from: the four input arrays (four scattered loads per
// list entry, each touching a cache line of its own), or the packed records of
// gsb_pack_gaussians (three 16-byte loads from one 48-byte record). Loads are unconditional in
// both, as in fetch_attrs.
template <bool kPacked> struct Attrs;
template <> struct Attrs<false> {
    const float2 *means;
    const F3 *conics;
    const float *opac;
    const F3 *colors;
    __device__ explicit Attrs(const ViewDesc &v)
        : means(reinterpret_cast<const float2 *>(v.means2d)),
          conics(reinterpret_cast<const F3 *>(v.conics)), opac(v.opacity),
          colors(reinterpret_cast<const F3 *>(v.colors)) {}
    __device__ GRaw fetch(uint32_t id, uint32_t n) const {
        return fetch_attrs(id, n, means, conics, opac, colors);
    }
};
template <> struct Attrs<true> {
    const float4 *rec;
    __device__ explicit Attrs(const ViewDesc &v) : rec(v.records) {}
    __device__ GRaw fetch(uint32_t id, uint32_t n) const {
        GRaw g;
        g.valid = id < n;
        g.id = g.valid ? id : 0u;
        const float4 *r = rec + 3 * size_t(g.id);
        const float4 a = r[0], b = r[1], c = r[2];
        g.x = a.x; g.y = a.y; g.A = a.z; g.B = a.w;
        g.C = b.x; g.o = b.y; g.r = b.z; g.g = b.w;
        g.b = c.x;
        return g;
    }
};

// Reach culling (plain form). A staged Gaussian cannot reach some quadrants of the tile:
// bit w of its mask is clear when no pixel of quadrant (w & 1, w >> 1) can have q >= kQCull, i.e.
// when the pair is skipped (alpha < 1/255) at every pixel of that quadrant. With Q the conic form
// of Eq. (power), q >= kQCull means Q(d) <= t, t = 2 (log2 o - kQCull) / log2 e, and the ellipse
// Q(d) <= t lies within |dx| <= sqrt(t Sxx), |dy| <= sqrt(t Syy) of the centre, with
// Sxx = C / det, Syy = A / det the covariance's diagonal (det = AC - B^2). The test is made
// conservative for the q the kernels compute: t is enlarged by a bound on its rounding error
// (taken as 2^-14 of the magnitudes of the terms it is formed from, far above the FP32 error of
// the per-pixel form), det is formed with the rounding error of B^2 recovered, and the
// half-widths get a relative and an absolute slack. A non-definite or non-finite conic (or a
// negative t) reaches every quadrant. (xh, yh) is the centre relative to the tile centre.
// A wavefront then skips, without evaluating q, the Gaussians that cannot reach its quadrant.
// Only the plain form uses it: there q costs a dozen instructions per pixel, while the GEMM form
// gets the q of a whole group from one product and skips a Gaussian with one compare.
struct Eval;
__device__ inline uint32_t reach_mask(const GRaw &g, const Eval &e);
__device__ inline uint32_t reach_mask(const GRaw &g, float lo2o, float xh, float yh) {
    const float gxh = fmaf(g.A, xh, g.B * yh), gyh = fmaf(g.C, yh, g.B * xh);
    const float Qh = fmaf(xh, gxh, yh * gyh);
    const float mag = kLog2e * (28.125f * (fabsf(g.A) + fabsf(g.C)) + 56.25f * fabsf(g.B) +
                                7.5f * (fabsf(gxh) + fabsf(gyh)) + 0.5f * fabsf(Qh)) + fabsf(lo2o);
    const float t = (lo2o - kQCull + fmaf(mag, 0x1p-14f, 0x1p-16f)) * (2.0f / kLog2e);
    const float bb = g.B * g.B;
    const float det = fmaf(g.A, g.C, -bb) - fmaf(g.B, g.B, -bb);
    if (!(det > 0.f)) return 0xfu;
    const float rdet = 1.0f / det;
    const float hx = fmaf(sqrtf(t * g.C * rdet), 1.0f + 0x1p-10f, fmaf(fabsf(xh), 0x1p-18f, 0x1p-6f));
    const float hy = fmaf(sqrtf(t * g.A * rdet), 1.0f + 0x1p-10f, fmaf(fabsf(yh), 0x1p-18f, 0x1p-6f));
    if (!(hx < 3.0e38f && hy < 3.0e38f)) return 0xfu;   // also NaN (A or C not positive, t < 0)
    // pixel columns (rows) of the tile are 0..15 relative to its corner; the centre is at 7.5
    const float xl = xh + 7.5f, yl = yh + 7.5f;
    const bool c0 = xl - hx <= 7.f && xl + hx >= 0.f, c1 = xl - hx <= 15.f && xl + hx >= 8.f;
    const bool r0 = yl - hy <= 7.f && yl + hy >= 0.f, r1 = yl - hy <= 15.f && yl + hy >= 8.f;
    return uint32_t(c0 && r0) | uint32_t(c1 && r0) << 1 | uint32_t(c0 && r1) << 2 |
           uint32_t(c1 && r1) << 3;
}

// What the staging of a list entry works out before it is written to LDS: the centre relative to the
// tile centre, log2 o (-inf for an entry that is never blended: alpha <= o < 1/255, or invalid), and
// g = Sigma^-1 (xh, yh) and Q there, to full FP32 accuracy.
struct Eval {
    bool live;
    float xh, yh, lo2o, gxh, gyh, Qh;
};
__device__ inline Eval evaluate(const GRaw &g, float xc, float yc) {
    Eval e;
    e.live = g.valid && g.o >= kTauCull;
    e.xh = g.x - xc;
    e.yh = g.y - yc;
    e.lo2o = e.live ? __log2f(g.o) : -INFINITY;
    e.Qh = quad_acc(g.A, g.B, g.C, e.xh, e.yh, e.gxh, e.gyh);
    return e;
}

__device__ inline uint32_t reach_mask(const GRaw &g, const Eval &e) {
    return reach_mask(g, e.lo2o, e.xh, e.yh);
}

// Whether a live entry can reach alpha >= 1/255 at a pixel of the tile; false only when the q that
// the kernels compute is below kQCull at all of them. Over the square of the pixel centres
// (7.5 px to each side of the tile centre) the smallest Q is 0 if the mean lies inside, else it lies
// on an edge that faces the mean: on the line dx = a (a the nearest dx of the square, 0 if the mean
// lies between its sides) at dy = -B a / C clamped to the square, or on dy = b likewise; the smaller
// of the two is the minimum, whichever edges face the mean. The entry is kept unless that minimum
// exceeds t, the level at which q = kQCull, enlarged by a bound on the error of the computed q (2^-14
// of the magnitudes of the terms that it is formed from, about eight times the BF16 form's error and
// far above the others') and of the minimum (2^-20 of its terms). Not a definite conic, a NaN or
// coefficients that the FP16 form clamps: kept. On the 4K frame this keeps 39% of a 3-sigma list's
// entries; the bounding box of the ellipse would keep 55%.
__device__ inline bool reaches_tile(const GRaw &g, const Eval &e) {
    const float mag = kLog2e * (28.125f * (fabsf(g.A) + fabsf(g.C)) + 56.25f * fabsf(g.B) +
                                7.5f * (fabsf(e.gxh) + fabsf(e.gyh)) + 0.5f * fabsf(e.Qh)) +
                      fabsf(e.lo2o);
    const float t = (e.lo2o - kQCull + fmaf(mag, 0x1p-14f, 0x1p-16f)) * (2.0f / kLog2e);
    const float bb = g.B * g.B;
    const float det = fmaf(g.A, g.C, -bb) - fmaf(g.B, g.B, -bb);
    const float a = e.xh - fminf(fmaxf(e.xh, -7.5f), 7.5f);
    const float b = e.yh - fminf(fmaxf(e.yh, -7.5f), 7.5f);
    const float v = fminf(fmaxf(-g.B * a * __builtin_amdgcn_rcpf(g.C), e.yh - 7.5f), e.yh + 7.5f);
    const float u = fminf(fmaxf(-g.B * b * __builtin_amdgcn_rcpf(g.A), e.xh - 7.5f), e.xh + 7.5f);
    const float s1 = fmaf(g.A * a, a, g.C * v * v), s2 = fmaf(g.C * b, b, g.A * u * u);
    constexpr float kLess = 1.0f - 0x1p-20f;
    const float q1 = fmaf(2.0f * g.B * a, v, s1 * kLess), q2 = fmaf(2.0f * g.B * b, u, s2 * kLess);
    const bool out = q1 > t && q2 > t && g.A > 0.f && g.C > 0.f && det > 0.f && mag < kF16Max;
    return !out;
}

// The 16-bit hi and lo terms of a live entry's coefficients (zeros otherwise) and the accumulator
// init.
template <Mode M>
__device__ inline void coefficients(const GRaw &g, const Eval &e, typename Op<M>::vec &ahi,
                                    typename Op<M>::vec &alo, float &kc) {
    float hi[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float lo[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float k0 = -INFINITY;
    if (e.live) {
        const float v[5] = {-0.5f * kLog2e * g.A, -0.5f * kLog2e * g.C, -kLog2e * g.B,
                            -kLog2e * e.gxh, -kLog2e * e.gyh};
        k0 = fmaf(e.Qh, -0.5f * kLog2e, e.lo2o);
#pragma unroll
        for (int k = 0; k < 5; ++k) hi[k] = v[k];
        const typename Op<M>::vec vh = Op<M>::cvt(hi);
#pragma unroll
        for (int k = 0; k < 5; ++k) lo[k] = (v[k] - Op<M>::back(vh, k)) * kLoScale;
    }
    ahi = Op<M>::cvt(hi);
    alo = Op<M>::cvt(lo);
    kc = k0;
}

// Which of a batch's entries are staged: those that can reach the tile (`all`: every one of the
// `len` entries of the batch, also those that are never blended). quad: the quadrants (wavefronts)
// that the entry can reach in the plain form.
template <Mode M>
__device__ inline bool keep_entry(const GRaw &g, const Eval &e, bool all, bool inside, uint32_t &quad) {
    bool keep = e.live && reaches_tile(g, e);
    quad = 0xfu;
    if constexpr (M == Mode::Plain) {
        quad = keep ? reach_mask(g, e) : 0u;
        keep = quad != 0u;
    }
    if (all) {
        keep = inside;
        quad = 0xfu;
    }
    return keep;
}

// Writes a kept entry into its slot (S: FwdStage or BwdStage).
template <Mode M, typename St>
__device__ inline void stage(const GRaw &g, const Eval &e, uint32_t quad, int slot, St &S) {
    if constexpr (M == Mode::Plain) {
        S.geo[slot] = e.live ? make_float4(g.x, g.y, g.A, g.B) : make_float4(0.f, 0.f, 0.f, 0.f);
        S.geo2[slot] = make_float2(e.live ? g.C : 0.f, e.lo2o);
        S.reach[slot] = uint8_t(quad);
    } else {
        typename Op<M>::vec ah, al;
        coefficients<M>(g, e, ah, al, S.kc[slot]);
        S.ahi[slot] = ah;
        S.alo[slot] = al;
    }
    S.attr[slot] = make_float4(e.lo2o, g.r, g.g, g.b);
}
// An open slot of the last group (GEMM form): q = -inf.
template <Mode M, typename St>
__device__ inline void stage_inert(int slot, St &S) {
    const float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    S.kc[slot] = -INFINITY;
    S.ahi[slot] = S.alo[slot] = Op<M>::cvt(z);
}

// ------------------------------------------------------------------------------- per-lane setup
struct Lane {
    int t, w, l;
    int col, row;            // pixel within tile
    float px, py;            // pixel coordinates
    bool inside;
    // MFMA A-operand read: which staged Gaussian of a group this lane supplies, if any
    bool a_valid;
    int a_g;
};

// kByCol: lane l holds pixel (l / 8, l % 8) of the quadrant instead of (l % 8, l / 8), which the
// backward's reduction needs (wave_grads).
template <bool kByCol>
__device__ inline Lane lane_setup(int tid, TileXY tile, int W, int H) {
    Lane L;
    L.t = tid; L.w = L.t >> 6; L.l = L.t & 63;
    // wave w owns the 8x8 quadrant (w & 1, w >> 1) of the tile: compact footprints touch fewer
    // waves than with 4-row strips, so fewer (Gaussian, wave) pairs have work
    L.col = 8 * (L.w & 1) + (kByCol ? L.l >> 3 : L.l & 7);
    L.row = 8 * (L.w >> 1) + (kByCol ? L.l & 7 : L.l >> 3);
    const int x0 = tile.x * kTile, y0 = tile.y * kTile;
    L.px = float(x0 + L.col); L.py = float(y0 + L.row);
    L.inside = (x0 + L.col < W) && (y0 + L.row < H);
    const int i = L.l & 31, h = L.l >> 5;
    L.a_valid = (h == ((i >> 2) & 1));
    L.a_g = 4 * (i >> 3) + (i & 3);
    return L;
}

template <Mode M>
__device__ inline void pixel_basis(const Lane &L, typename Op<M>::vec &bhi, typename Op<M>::vec &blo) {
    if constexpr (M != Mode::Plain) {
        const float xb = 7.5f - float(L.col), yb = 7.5f - float(L.row);
        float v[8] = {xb * xb, yb * yb, xb * yb, xb, yb, 0.f, 0.f, 0.f};
        bhi = Op<M>::cvt(v);
        float s[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k] = v[k] * kLoScaleInv;
        blo = Op<M>::cvt(s);
    }
}

// q of the 16 staged Gaussians from slot s0: one value per register, from the accumulator init and
// the two A operands.
template <Mode M>
__device__ inline f16x group_q(const float *kc, const typename Op<M>::vec &ah,
                               const typename Op<M>::vec &al, const typename Op<M>::vec &bhi,
                               const typename Op<M>::vec &blo) {
    f16x acc;
    const float4 *kc4 = reinterpret_cast<const float4 *>(kc);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float4 k = kc4[j];
        acc[4 * j + 0] = k.x; acc[4 * j + 1] = k.y; acc[4 * j + 2] = k.z; acc[4 * j + 3] = k.w;
    }
    acc = Op<M>::mfma(ah, bhi, acc);
    return Op<M>::mfma(al, blo, acc);
}
// Forward: the operands through a select per operand, which holds fewer registers than the
// backward's one pointer (8 wavefronts per SIMD).
template <Mode M, int NB>
__device__ inline f16x group_q(const FwdStage<M, NB> &S, int s0, const Lane &L,
                               const typename Op<M>::vec &bhi, const typename Op<M>::vec &blo) {
    return group_q<M>(&S.kc[s0], *(L.a_valid ? &S.ahi[s0 + L.a_g] : &S.zero),
                      *(L.a_valid ? &S.alo[s0 + L.a_g] : &S.zero), bhi, blo);
}
// Backward: one address per lane. A lane off the diagonal reads zero_hi and zero_lo whatever s0 is
// (its step is 0), and every lane's lo operand lies at one fixed offset from its hi operand, so the
// lo read takes no address arithmetic of its own (the selects depend on the lane only and leave the
// loops): one vector instruction per group instead of five.
template <Mode M, int NB>
__device__ inline f16x group_q(const BwdStage<M, NB> &S, int s0, const Lane &L,
                               const typename Op<M>::vec &bhi, const typename Op<M>::vec &blo) {
    typedef typename Op<M>::vec vec;
    typedef BwdStage<M, NB> St;
    const vec *base = L.a_valid ? &S.ahi[L.a_g] : &S.zero_hi;
    const int step = L.a_valid ? 1 : 0;
    const vec *ph = base + s0 * step;
    // (the same distance for every slot: zero_hi follows ahi as zero_lo follows alo)
    const ptrdiff_t lo_off = reinterpret_cast<const char *>(&S.zero_lo) -
                             reinterpret_cast<const char *>(&S.zero_hi);
    static_assert(sizeof(St::ahi) == sizeof(St::alo), "zero_lo must mirror zero_hi");
    return group_q<M>(&S.kc[s0], *ph,
                      *reinterpret_cast<const vec *>(reinterpret_cast<const char *>(ph) + lo_off),
                      bhi, blo);
}

// Plain form: which of the 16 staged Gaussians from slot s0 (below `total`) can reach the
// wavefront's quadrant.
template <typename St>
__device__ inline uint32_t group_reach(const St &S, int s0, int total, const Lane &L) {
    const int u = L.l & (kGroup - 1);
    const uint32_t r = s0 + u < total ? S.reach[s0 + u] : 0u;
    return uint32_t(__builtin_amdgcn_ballot_w64(((r >> L.w) & 1u) != 0u)) & 0xffffu;
}
__device__ inline uint32_t uniform(uint32_t x) { return uint32_t(__builtin_amdgcn_readfirstlane(int(x))); }

// q of one staged Gaussian for this lane's pixel, per pixel in FP32 (Eq. (power)).
__device__ inline float plain_q(const float4 &geo, const float2 &g2, const Lane &L) {
    const float dx = geo.x - L.px, dy = geo.y - L.py;
    float gx, gy;
    return fmaf(quad_acc(geo.z, geo.w, g2.x, dx, dy, gx, gy), -0.5f * kLog2e, g2.y);
}

// ------------------------------------------------------------------------------- forward
struct FwdState {
    float T, r, g, b, thr;   // thr = kQCull while live, +inf once done
    // 1-based list position of the last blended entry; ~slot for one blended in this batch, until
    // the batch ends
    int last;
};

// One front-to-back step (Alg. 1 / Alg. 2 inner loop) for this lane's pixel: a skipped pair or a
// finished pixel leaves the state unchanged. The kernel is bound by vector-instruction issue, so
// the lanes that blend update their state under the execution mask rather than through a select
// per value. (The end of a pixel stays a select: as a scalar branch on a ballot it costs more
// than it saves, since the branch waits for the compare.)
__device__ inline void composite(float q, float lo2o, float cr, float cg, float cb, int slot,
                                 FwdState &st) {
    const bool hit = q >= st.thr;
    const float a = __builtin_amdgcn_exp2f(fminf(fminf(q, lo2o), kQAlphaMax));   // <= 0.99
    const float Tn = fmaf(-a, st.T, st.T);   // T (1 - alpha), rounded once
    const bool stop = Tn < kTStop;
    if (hit && !stop) {
        const float wgt = a * st.T;
        st.r = fmaf(wgt, cr, st.r);
        st.g = fmaf(wgt, cg, st.g);
        st.b = fmaf(wgt, cb, st.b);
        st.T = Tn;
        st.last = ~slot;
    }
    st.thr = (hit && stop) ? INFINITY : st.thr;
}

// Composites the 16 Gaussians of one group; q(u) gives Gaussian u's exponent for this lane. A
// Gaussian that some lane takes has its (log2 o, r, g, b) read at one LDS address by every lane.
// A Gaussian whose bit in `reach` (this wavefront's reach mask of the group) is clear is skipped
// without evaluating q: no lane would take it.
// kFew (see few_tiles): the whole group's values are read ahead, into registers.
template <bool kFew, typename QFn>
__device__ inline void composite_group(const float4 *attr, int base, uint32_t reach, FwdState &st,
                                       QFn q_of) {
    f4x ahead[kFew ? kGroup : 1];
    if constexpr (kFew) {
#pragma unroll
        for (int u = 0; u < kGroup; ++u) ahead[u] = *reinterpret_cast<const f4x *>(&attr[u]);
#pragma unroll
        for (int u = 0; u < kGroup; ++u) asm volatile("" : "+v"(ahead[u]));
    }
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
        if (((reach >> u) & 1u) == 0u) continue;
        const float q = q_of(u);
        if (__builtin_amdgcn_ballot_w64(q >= st.thr) == 0ull) continue;   // no lane takes it
        // one address for every lane (an LDS broadcast), read whole: left to itself the compiler
        // moves the colour reads into the blending lanes' branch, as separate loads
        f4x a = kFew ? ahead[kFew ? u : 0] : *reinterpret_cast<const f4x *>(&attr[u]);
        if constexpr (!kFew) asm volatile("" : "+v"(a));
        composite(q, a.x, a.y, a.z, a.w, base + u, st);
    }
}

// Forward of one tile of one view (all 256 threads of the block take part; block-uniform control
// flow around every barrier).
// kAll: every entry is staged in its own place, as v.reach = 0 asks (the caller has looked at it), with no
// test and no count, in two buffers in turn with one barrier a batch: GSB_FULL_SCAN's forward (FP32, 4K
// frame of 3M Gaussians: as a selection that keeps everything 1217 us, this 1135; 1 M at 1080p 397 and 365).
template <bool kAll> constexpr int kFwdBuffers = kAll ? 2 : 1;
constexpr int kAllBatchFwd = 128;
template <Mode M, int NB, bool kPacked = false, bool kFew = false, bool kAll = false>
__device__ inline void fwd_tile(const ViewDesc &v, TileXY tile, FwdStage<M, NB> (&stages)[kFwdBuffers<kAll>],
                                int tid = threadIdx.x) {
    static_assert(NB % kGroup == 0 && NB <= kBlock, "batch must be whole groups, <= block");
    const uint32_t *plist = v.point_list;
    const uint32_t n = uint32_t(v.n);
    const Attrs<kPacked> src(v);
    const Lane L = lane_setup<false>(tid, tile, v.W, v.H);
    const float xc = float(tile.x * kTile) + 7.5f, yc = float(tile.y * kTile) + 7.5f;
    typename Op<M>::vec bhi, blo;
    pixel_basis<M>(L, bhi, blo);
    if (L.t == 0) {
        float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if constexpr (M != Mode::Plain) {
            for (FwdStage<M, NB> &S : stages) S.zero = Op<M>::cvt(z);
        }
    }
    uint2 rg = reinterpret_cast<const uint2 *>(v.ranges)[tile.y * v.gx + tile.x];
    // (the same in every lane, which the compiler does not see in a plan's kernels: their loops over batches
    // and groups ran on vector registers, 1 M Gaussians at 1080p in batches of 128 196 us, now 185)
    rg = make_uint2(uniform(rg.x), uniform(rg.y));
    // without Gaussians every list entry would be invalid: the tile shows the background
    const int64_t start = rg.x, len = n == 0 ? 0 : int64_t(rg.y) - int64_t(rg.x);
    const int nb = int((len + NB - 1) / NB);

    // list entries are loaded two batches ahead and attributes one batch ahead, so that neither
    // load waits on the other within an iteration
    const auto entry = [&](int bb) {          // batch bb's entry for this thread (bb < nb + 2)
        const int64_t o = int64_t(bb) * NB + L.t;
        return load_entry(plist, start + o, L.t < NB && o < len, start);
    };
    FwdState st{1.f, 0.f, 0.f, 0.f, L.inside ? kQCull : INFINITY, 0};
    GRaw nxt{};
    Entry ent{kNoEntry, false};
    if (nb > 0) {                               // (len > 0, so entry `start` exists)
        nxt = src.fetch(entry(0).id(), n);
        ent = entry(1);
    }
    for (int b = 0; b < nb; ++b) {
        const int base = b * NB;
        // Of the batch's entries only those that can reach the tile are staged, in order: a wavefront
        // posts how many it keeps and whether it still has a live pixel; the block leaves once none
        // has. (v.reach 0: every entry is staged, also those that are never blended.)
        const Eval e = evaluate(nxt, xc, yc);
        FwdStage<M, NB> &S = stages[kAll ? b & 1 : 0];
        const bool inside = L.t < NB && base + L.t < len;
        uint32_t quad = 0xfu;
        bool keep = inside;
        if constexpr (!kAll) keep = keep_entry<M>(nxt, e, v.reach == 0, inside, quad);
        const unsigned long long kept = kAll ? 0ull : __builtin_amdgcn_ballot_w64(keep);
        int total = len - base < NB ? int(len - base) : NB;
        if constexpr (kAll) {
            if (keep) stage<M>(nxt, e, quad, L.t, S);
            if constexpr (M != Mode::Plain) {
                if (total + L.t < (total + kGroup - 1) / kGroup * kGroup) stage_inert<M>(total + L.t, S);
            }
        }
        const bool wave_live = __ballot(st.thr != INFINITY) != 0;   // (the whole wavefront's)
        if (L.l == 0) S.post[L.w] = uint32_t(__popcll(kept)) + (wave_live ? kWaveLive : 0u);
        __syncthreads();             // every wavefront is done with the last batch
        const uint4 f = *reinterpret_cast<const uint4 *>(S.post);
        const uint32_t p[4] = {uniform(f.x), uniform(f.y), uniform(f.z), uniform(f.w)};
        const uint32_t all = p[0] + p[1] + p[2] + p[3];
        if (all < kWaveLive) break;
        if constexpr (!kAll) {
            total = int(all & (kWaveLive - 1));
            if (keep) {
                uint32_t before = 0;
#pragma unroll
                for (int k = 0; k < 3; ++k) before += k < L.w ? p[k] & (kWaveLive - 1) : 0u;
                const int slot = int(__builtin_amdgcn_mbcnt_hi(
                    uint32_t(kept >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(kept), before)));
                stage<M>(nxt, e, quad, slot, S);
                S.pos[slot] = uint8_t(L.t);
            }
            if constexpr (M != Mode::Plain) {      // the last group's open slots: q = -inf
                if (total + L.t < (total + kGroup - 1) / kGroup * kGroup) stage_inert<M>(total + L.t, S);
            }
            __syncthreads();
        }
        const int ng = (total + kGroup - 1) / kGroup;
        // unconditional: past the last batch these read entry `start` and Gaussian 0, unused
        nxt = src.fetch(ent.id(), n);
        ent = entry(b + 2);
        for (int g = 0; g < ng; ++g) {
            if (__ballot(st.thr != INFINITY) == 0) break;
            const int s0 = g * kGroup;
            const float4 *attr = &S.attr[s0];
            const auto reach = [&] {
                if constexpr (M == Mode::Plain && !kAll) return group_reach(S, s0, total, L);
                return total - s0 >= kGroup ? 0xffffu : (1u << (total - s0)) - 1u;
            };
            if constexpr (M == Mode::Plain && kFew) {
                f4x geo[kGroup];
                float2 geo2[kGroup];
#pragma unroll
                for (int k = 0; k < kGroup; ++k) {
                    geo[k] = *reinterpret_cast<const f4x *>(&S.geo[s0 + k]);
                    geo2[k] = S.geo2[s0 + k];
                }
#pragma unroll
                for (int k = 0; k < kGroup; ++k) {
                    asm volatile("" : "+v"(geo[k]));
                    asm volatile("" : "+v"(geo2[k].x), "+v"(geo2[k].y));
                }
                composite_group<kFew>(attr, s0, reach(), st, [&](int k) {
                    return plain_q(make_float4(geo[k].x, geo[k].y, geo[k].z, geo[k].w), geo2[k], L);
                });
            } else if constexpr (M == Mode::Plain) {
                composite_group<kFew>(attr, s0, reach(), st,
                                      [&](int k) { return plain_q(S.geo[s0 + k], S.geo2[s0 + k], L); });
            } else {
                const f16x q = group_q<M, NB>(S, s0, L, bhi, blo);
                composite_group<kFew>(attr, s0, 0xffffu, st, [&](int k) { return q[k]; });
            }
        }
        if (st.last < 0) st.last = base + (kAll ? ~st.last : int(S.pos[~st.last])) + 1;
    }
    if (L.inside) {
        const int64_t p = int64_t(L.py) * v.W + int64_t(L.px);
        const int64_t HW = int64_t(v.H) * v.W;
        v.image[p] = st.r + st.T * v.bg[0];
        v.image[HW + p] = st.g + st.T * v.bg[1];
        v.image[2 * HW + p] = st.b + st.T * v.bg[2];
        v.final_T[p] = st.T;
        v.last_contrib[p] = st.last;
    }
}

// ------------------------------------------------------------------------------- backward
// u + (v moved within its 16-lane row by the DPP control Ctrl). Every control used here reads
// inside the row, so bound_ctrl (out-of-row reads give 0) never applies; it spares an `old`
// operand.
template <int Ctrl>
__device__ inline float dpp_add2(float u, float v) {
    const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(v), Ctrl, 0xf, 0xf, true);
    return u + __int_as_float(y);
}
constexpr int kDppRowRor8 = 0x128, kDppRowHalfMirror = 0x141;
constexpr int kDppQuadRev = 0x1b, kDppQuadSwap = 0xb1;       // quad_perm [3,2,1,0], [1,0,3,2]

// The wavefront is halved for a pair of values at a time: permlane32_swap + add leaves the first
// value's 32 partial sums in lanes 0-31 and the second's in lanes 32-63, permlane16_swap + add does
// the same on 16-lane rows. Every lane must be active.
__device__ inline float swap_add32(float &x, float y) {   // returns [x.lo + x.hi | y.lo + y.hi]
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float swap_add16(float x, float y) {    // rows: [x0+x1, y0+y1, x2+x3, y2+y3]
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The nine gradient sums of one Gaussian over the wavefront's 8x8 pixels, with lane l at column
// l / 8 and row l % 8 (Lane<kByCol>). The geometric terms are separable, dL/dpower dx^i dy^j, so
// only six values per lane are summed over the columns (three levels of swaps): g0 = dL/dpower,
// g0 dx, g0 dx^2 and the three colours. The eight slots of 8 lanes that these leave in one register
// hold each row's six sums, and g0 and g0 dx a second time, which the row's dy then turns into the
// terms of S_y and S_xy, and g0 dy once more into S_yy; three more levels add the rows. 24 vector
// instructions (the products by dx and dy included) against 29, and two LDS crossbar operations,
// for nine values formed per pixel and summed over all six levels; the 4K BF16 backward 2.49 -> 2.25
// ms with one compare for both clamps.
//   a: rows (16 lanes) g0, g0 dx^2, g0 dx, colour r;  b: rows colour g, g0, colour b, g0 dx;
//   a and b share one register: lanes 0-7 of a row take a's, lanes 8-15 b's.
// Result: lane l with l % 8 == 0 and lane 28 hold the word sum_word(l) of the Gaussian's sums.
__device__ inline float wave_grads(float g0, float dx, float dy, float cr, float cg, float cb,
                                   int lane) {
    const float g1 = g0 * dx;
    float x0 = g0, x2 = g1 * dx, x4 = cg;
    const float p0 = swap_add32(x0, g1), p1 = swap_add32(x2, cr), p2 = swap_add32(x4, cb);
    const float a = swap_add16(p0, p1), b = swap_add16(p2, p0);
    const bool lo8 = (lane & 8) == 0, lo4 = (lane & 4) == 0, by_dy = (lane & 24) == 24;
    float s = dpp_add2<kDppRowRor8>(lo8 ? a : b, lo8 ? b : a);
    s *= by_dy ? dy : 1.0f;
    const float t = s * dy;
    s = dpp_add2<kDppRowHalfMirror>(lo4 ? s : t, lo4 ? t : s);
    s = dpp_add2<kDppQuadRev>(s, s);
    s = dpp_add2<kDppQuadSwap>(s, s);
    // keep the last add here, where it is one DPP add, not moved into the callers' leader branch
    // (where it would need a separate move)
    asm volatile("" : "+v"(s));
    return s;
}

// The word of a Gaussian's nine sums (S_xx, S_xy, S_yy, S_x, S_y, S, r, g, b) that a leader lane
// (l % 8 == 0, or 28) holds after wave_grads.
__device__ inline bool sum_leader(int l) { return (l & 7) == 0 || l == 28; }
__device__ inline int sum_word(int l) {
    // 8-lane group l / 8: S, g, S_xx, S_y, S_x, b, r, S_xy
    return l == 28 ? 2 : int((0x16834075u >> (4 * (l >> 3))) & 15u);
}

// Sum of 9 values over the whole wavefront (the deterministic gather's lane sums), transposed so
// that the 9 totals land in distinct lanes: lanes 16r .. 16r+7 of ab hold s[{0,2,1,3}[r]], lanes
// 16r+8 .. 16r+15 hold s[4 + {0,2,1,3}[r]]; lanes 0-7 of c hold s8 (whose first two levels go
// through the LDS crossbar). Every lane must be active.
__device__ inline void wave_sum9(const float (&s)[kGrad], int lane, float &ab, float &c) {
    float x0 = s[0], x2 = s[2], x4 = s[4], x6 = s[6];
    const float p01 = swap_add32(x0, s[1]), p23 = swap_add32(x2, s[3]);
    const float p45 = swap_add32(x4, s[5]), p67 = swap_add32(x6, s[7]);
    const float p88 = s[8] + __int_as_float(__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2,
                                                                        __float_as_int(s[8])));
    const float a = swap_add16(p01, p23);
    const float b = swap_add16(p45, p67);
    c = p88 + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(p88), 0x401f));
    const bool lo = (lane & 8) == 0;
    ab = dpp_add2<kDppRowRor8>(lo ? a : b, lo ? b : a);
    c = dpp_add2<kDppRowRor8>(c, c);
    ab = dpp_add2<kDppRowHalfMirror>(ab, ab); c = dpp_add2<kDppRowHalfMirror>(c, c);
    ab = dpp_add2<kDppQuadRev>(ab, ab);       c = dpp_add2<kDppQuadRev>(c, c);
    ab = dpp_add2<kDppQuadSwap>(ab, ab);      c = dpp_add2<kDppQuadSwap>(c, c);
}

struct BwdState {
    float T;        // transmittance in front of the pairs not yet visited
    // the colour behind them per unit of that transmittance: (T_final (bg . g) + sum over the
    // visited pairs of alpha T (c . g)) / T. With it dL/dalpha of the next pair (in front) is
    // T_in (c . g - beta), T_in the transmittance in front of that pair, and beta moves to
    // beta (1 - alpha) + alpha (c . g): no division by (1 - alpha) beyond the one T needs.
    float beta;
    float gr, gg, gb;
    int last;
};

// Reverse step for one (Gaussian, pixel) pair. Nothing but a compare and a scalar branch is
// spent when no lane of the wave has a live pair. Otherwise every lane evaluates the step, with no
// branch but a rare one for the clamps (a dead lane takes alpha = 0: its terms vanish and its
// state is unchanged exactly, since 1 / (1 - 0) = 1),
// the pair's 9 gradient terms are summed over the wavefront (wave_grads), and the totals are added
// into the Gaussian's LDS accumulator (`acc` points at the word this lane adds when it leads, see
// sum_word), which the block flushes to global memory once per batch. Raw
// sums: S_xx, S_xy, S_yy, S_x, S_y (times dL/dpower), the sum of dL/dpower without the clamp test
// (o dL/do: the final pass divides it by o, once per Gaussian instead of once per pair), and the
// three colour gradients.
// kRanged = false: the caller has checked that the whole group lies before every lane's last
// contributor, so the skip test alone decides (one compare, whose mask is the ballot).
// In the deterministic backward `acc` points into the wavefront's own slice of the batch's sums
// (zero before; no other wavefront adds there, so the sum has a fixed order).
template <bool kRanged>
__device__ inline void reverse_pair(float q, bool in_range, const float4 *ga, const float2 *gb,
                                    int u, const Lane &L, BwdState &st, float *acc) {
    bool alive;
    unsigned long long live;
    if constexpr (kRanged) {
        // one ballot per compare (each is just that compare's lane mask), combined and tested in
        // scalar registers: a ballot of the combined condition is copied through a vector
        // register, two more vector instructions for every Gaussian of a ranged group. The empty
        // asm statements keep the compiler from merging the two ballots back into one, and the
        // lane's own condition is read back from the combined mask (with the compares reused,
        // each mask is copied beside its ballot: two scalar moves per visit).
        unsigned long long m_range = __builtin_amdgcn_ballot_w64(in_range);
        unsigned long long m_cull = __builtin_amdgcn_ballot_w64(q >= kQCull);
        asm volatile("" : "+s"(m_range));
        asm volatile("" : "+s"(m_cull));
        live = m_range & m_cull;
        alive = __builtin_amdgcn_inverse_ballot_w64(live);
    } else {
        alive = q >= kQCull;
        live = __builtin_amdgcn_ballot_w64(alive);
    }
    if (live == 0ull) return;
    const float4 attr = ga[u];   // one address for every lane: LDS broadcasts
    const float2 bw = gb[u];
    // a dead lane has q < log2(1/255) or is past its last contributor: it blended nothing here.
    // (The clamp at the lowest argument that gives 0.99f, so that an exponent the minimum cut,
    // q > m, is the one test for both clamps: the same alpha bit for bit.)
    const float m = fminf(fminf(q, attr.x), kQAlphaMaxLo);
    const float a = alive ? __builtin_amdgcn_exp2f(m) : 0.f;
    const float r = __builtin_amdgcn_rcpf(1.0f - a);  // exactly 1 for a dead lane
    const float Tb = st.T * r;                           // T in front of this Gaussian
    const float wc = a * Tb;                             // the pair's weight alpha T
    // c . g - beta as one fma chain from -beta: dL/dalpha = Tb (c . g - beta)
    const float gmb = fmaf(st.gb, attr.w, fmaf(st.gg, attr.z, fmaf(st.gr, attr.y, -st.beta)));
    st.beta = fmaf(a, gmb, st.beta);
    st.T = Tb;
    float da = wc * gmb;                                 // dL/dpower = alpha dL/dalpha
    // The clamps are rare, so one scalar test stands for them and the terms of the live lanes they
    // touch are zeroed in place: with the 0.99 clamp active dL/dpower is 0, and no gradient
    // reaches the geometry through a clamped (positive) power.
    if ((__builtin_amdgcn_ballot_w64(q > m) & live) != 0ull) {
        const bool keep_a = !(q > kQAlphaMaxLo && attr.x > kQAlphaMaxLo);
        const bool keep_g = keep_a && !(q > attr.x);
        // a clamped power still passes its gradient to the opacity (dL/do = alpha/o dL/dalpha):
        // those lanes' part of that sum is added here, apart from the geometry's
        float e = keep_a && !keep_g ? da : 0.f;
        da = keep_g ? da : 0.f;
        e = swap_add32(e, e);
        e = swap_add16(e, e);
        e = dpp_add2<kDppRowRor8>(e, e);
        e = dpp_add2<kDppRowHalfMirror>(e, e);
        e = dpp_add2<kDppQuadRev>(e, e);
        e = dpp_add2<kDppQuadSwap>(e, e);
        if (L.l == 0) atomicAdd(acc, e);                 // lane 0's word is the opacity sum
    }
    const float dx = bw.x - L.px, dy = bw.y - L.py;
    const float sum = wave_grads(da, dx, dy, wc * st.gr, wc * st.gg, wc * st.gb, L.l);
    // one LDS atomic for all nine sums
    if (sum_leader(L.l)) atomicAdd(acc, sum);
}

// Sum of 4 values over the wavefront (two value pairs share each swap): lanes 16r ..
// 16r + 15 of the result hold s[{0,2,1,3}[r]]. Every lane must be active.
__device__ inline float wave_sum4(const float (&s)[4]) {
    float x0 = s[0], x2 = s[2];
    const float p01 = swap_add32(x0, s[1]), p23 = swap_add32(x2, s[3]);
    float a = swap_add16(p01, p23);
    a = dpp_add2<kDppRowRor8>(a, a);
    a = dpp_add2<kDppRowHalfMirror>(a, a);
    a = dpp_add2<kDppQuadRev>(a, a);
    a = dpp_add2<kDppQuadSwap>(a, a);
    return a;
}

// Reverse step of reverse_pair for the matrix-core reduction: the same state update, but of the
// pair's gradient terms only the four plain sums (dL/do and the colours) are reduced on the vector
// ALUs here; dL/dpower (with no gradient through a clamped power) goes into the wavefront's
// transposition row `dgrow`, from which the five geometric sums are formed as a product with the
// pixel basis (mm_reduce). Returns whether any lane of the wavefront had a live pair.
template <bool kRanged>
__device__ inline bool reverse_pair_mm(float q, bool in_range, const float4 *ga, const float2 *gb,
                                       int u, const Lane &L, BwdState &st, float *acc,
                                       uint32_t *dgrow) {
    bool alive;
    unsigned long long live;
    if constexpr (kRanged) {
        unsigned long long m_range = __builtin_amdgcn_ballot_w64(in_range);
        unsigned long long m_cull = __builtin_amdgcn_ballot_w64(q >= kQCull);
        asm volatile("" : "+s"(m_range));
        asm volatile("" : "+s"(m_cull));
        live = m_range & m_cull;
        alive = __builtin_amdgcn_inverse_ballot_w64(live);
    } else {
        alive = q >= kQCull;
        live = __builtin_amdgcn_ballot_w64(alive);
    }
    if (live == 0ull) return false;
    const float4 attr = ga[u];
    const float araw = __builtin_amdgcn_exp2f(fminf(q, attr.x));
    const float a = alive ? fminf(araw, kAlphaMax) : 0.f;
    const float r = __builtin_amdgcn_rcpf(1.0f - a);
    const float Tb = st.T * r;
    const float wc = a * Tb;
    const float gmb = fmaf(st.gb, attr.w, fmaf(st.gg, attr.z, fmaf(st.gr, attr.y, -st.beta)));
    st.beta = fmaf(a, gmb, st.beta);
    st.T = Tb;
    const float da = araw < kAlphaMax ? wc * gmb : 0.f;
    const float dg = q > attr.x ? 0.f : da;
    // dg = hi + lo 2^-12 with FP16 hi and lo (truncations; the residual dg - hi is exact in FP32)
    const auto hp = __builtin_amdgcn_cvt_pkrtz(dg, 0.f);
    const float lo = (dg - float(hp[0])) * kLoScale;
    const auto pk = __builtin_amdgcn_cvt_pkrtz(dg, lo);
    dgrow[L.l] = __builtin_bit_cast(uint32_t, pk);
    const float s[4] = {da, wc * st.gr, wc * st.gg, wc * st.gb};
    const float tot = wave_sum4(s);
    if ((L.l & 15) == 0)
        atomicAdd(acc + 5 + ((L.l >> 4) == 1 ? 2 : (L.l >> 4) == 2 ? 1 : (L.l >> 4)), tot);
    return true;
}

// The pixel basis of the matrix-core reduction as the B operand of v_mfma_f32_16x16x32_f16, for
// the two 32-pixel halves c of the wavefront's quadrant: lane l supplies basis function l % 16
// (1, xb, yb, xb^2, xb yb, yb^2, then zeros) at the 8 pixels 32c + 8(l / 16) + j, j = 0..7, which
// lie in one row of the quadrant. xb = x_c - px and yb = y_c - py are quarter-integers of at most
// 7.5 in magnitude, so every value is exact in FP16.
__device__ inline void mm_basis(const Lane &L, h8 (&B)[2]) {
    const int n = L.l & 15;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float yb = 7.5f - float(8 * (L.w >> 1) + 4 * c + (L.l >> 4));
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float xb = 7.5f - float(8 * (L.w & 1) + j);
            v[j] = n == 0 ? 1.f : n == 1 ? xb : n == 2 ? yb : n == 3 ? xb * xb
                 : n == 4 ? xb * yb : n == 5 ? yb * yb : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) B[c][j] = _Float16(v[j]);
    }
}

// The five geometric sums of the 8 Gaussians of one half-group (staged slots base .. base + 7)
// from the wavefront's transposition rows: two v_mfma_f32_16x16x32_f16 give, per Gaussian, the
// moments sum_p dg [1, xb, yb, xb^2, xb yb, yb^2] over the 64 pixels (rows 0-7 from the hi terms,
// rows 8-15 from the lo terms, combined in FP32); with dx = xh + xb (xh = x - x_c) the sums
// of dg [dx^2, dx dy, dy^2, dx, dy] follow per Gaussian, and are added into the batch's
// accumulator. `hmask` has bit i set when Gaussian base + i had a live pair in this wavefront;
// the rows are left zero.
__device__ inline void mm_reduce(uint32_t (*rows)[kDgStride], const h8 (&B)[2], unsigned hmask,
                                 const float2 *gb, float xc, float yc, float *acc, const Lane &L) {
    __builtin_amdgcn_wave_barrier();
    const int row = L.l & 15, q = L.l >> 4;
    // hi rows take the low halves of the packed words, lo rows the high halves
    const uint32_t sel = row < 8 ? 0x05040100u : 0x07060302u;
    f4x d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const uint4 *src = reinterpret_cast<const uint4 *>(&rows[row & 7][32 * c + 8 * q]);
        const uint4 w0 = src[0], w1 = src[1];
        uint32_t av[4];
        av[0] = __builtin_amdgcn_perm(w0.y, w0.x, sel);
        av[1] = __builtin_amdgcn_perm(w0.w, w0.z, sel);
        av[2] = __builtin_amdgcn_perm(w1.y, w1.x, sel);
        av[3] = __builtin_amdgcn_perm(w1.w, w1.z, sel);
        h8 A;
        __builtin_memcpy(&A, av, sizeof(A));
        d = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, B[c], d, 0, 0, 0);
    }
    // lane l < 32 holds rows 4q + v (hi) of column l % 16; lane l + 32 the lo rows of the same
    // Gaussians: moment = hi + 2^-12 lo
    float m[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[v]), __float_as_uint(d[v]),
                                                        false, false);
        m[v] = fmaf(__uint_as_float(r[1]), kLoScaleInv, __uint_as_float(r[0]));
    }
    // moments table mom[g][n] in row 0 (the operand reads above have completed: the MFMA used them)
    float *mom = reinterpret_cast<float *>(rows[0]);
    if (L.l < 32 && row < 6) {
#pragma unroll
        for (int v = 0; v < 4; ++v) mom[(4 * q + v) * 8 + row] = m[v];
    }
    __builtin_amdgcn_wave_barrier();
    // lane g * 5 + k forms sum k of Gaussian g
    if (L.l < 40) {
        const int g = L.l / 5, k = L.l - 5 * g;
        if ((hmask >> g) & 1u) {
            const float4 m0 = *reinterpret_cast<const float4 *>(mom + 8 * g);
            const float2 m1 = *reinterpret_cast<const float2 *>(mom + 8 * g + 4);
            const float S1 = m0.x, Sx = m0.y, Sy = m0.z, Sxx = m0.w, Sxy = m1.x, Syy = m1.y;
            const float2 bw = gb[g];
            const float xh = bw.x - xc, yh = bw.y - yc;
            const float sx = fmaf(xh, S1, Sx), sy = fmaf(yh, S1, Sy);
            float val;
            if (k == 0) val = fmaf(xh, sx, fmaf(xh, Sx, Sxx));            // sum dg dx^2
            else if (k == 1) val = fmaf(xh, sy, fmaf(yh, Sx, Sxy));       // sum dg dx dy
            else if (k == 2) val = fmaf(yh, sy, fmaf(yh, Sy, Syy));       // sum dg dy^2
            else if (k == 3) val = sx;
            else val = sy;
            atomicAdd(acc + g * kGrad + k, val);
        }
    }
    __builtin_amdgcn_wave_barrier();
    // leave the rows zero for the next half-group
    uint4 *z = reinterpret_cast<uint4 *>(&rows[L.l >> 3][(L.l & 7) * 8]);
    z[0] = make_uint4(0u, 0u, 0u, 0u);
    z[1] = make_uint4(0u, 0u, 0u, 0u);
}

// Backward of one tile of one view.
// kMM: the five geometric sums are formed on the matrix cores (mm_reduce) instead of being
// reduced on the vector ALUs with the other four; `mm` is then the block's transposition tiles.
// The list entries that the backward takes at a time, of the NB that LDS has room for: a tile whose list
// is one batch loads, stages, blends and flushes one after the other, so short lists are taken in
// smaller batches, whose loads and flushes overlap the blending. Long lists, of which fewer entries
// are kept, fill the groups better in large ones. Backward in us with batches of 64, 128, 256, by the
// list's mean length: 246 entries 1739, 1835, 2233; 348: 839, 851, 933; 641: 1918, 1890, 2005;
// 1689: 2275, 2055, 1975. With this rule 1724, 850, 1892 and 1968.
template <int NB>
__device__ inline int batch_bwd(int64_t len) {
    if (NB >= 128 && len <= 256) return 64;
    if (NB > 128 && len <= 512) return 128;
    return NB;
}
// kDet: the batch sums go to the wavefronts' own slices (`det`) instead of `acc_`, and the flush
// writes the nine sums of each list position that has a nonzero one to the position's row in place of
// the global atomics.
template <Mode M, int NB, bool kMM, bool kPacked = false, bool kDet = false>
__device__ inline void bwd_tile(const ViewDesc &v, TileXY tile, BwdStage<M, NB> &S,
                                BwdAcc<NB> *acc_, int &s_maxlast, BwdMM *mm,
                                BwdAccDet<NB> *det = nullptr, int tid = threadIdx.x) {
    static_assert(NB % kGroup == 0 && NB <= kBlock, "batch must be whole groups, <= block");
    static_assert(!(kMM && kDet), "the deterministic backward reduces on the vector ALUs");
    const uint32_t *plist = v.point_list;
    const uint32_t n = uint32_t(v.n);
    const Attrs<kPacked> src(v);
    const Lane L = lane_setup<!kMM>(tid, tile, v.W, v.H);
    const int word = sum_word(L.l);   // the sum this lane adds when it leads a reduction
    const float xc = float(tile.x * kTile) + 7.5f, yc = float(tile.y * kTile) + 7.5f;
    typename Op<M>::vec bhi, blo;
    pixel_basis<M>(L, bhi, blo);
    if (L.t == 0) {
        float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if constexpr (M != Mode::Plain) S.zero_hi = S.zero_lo = Op<M>::cvt(z);
        s_maxlast = 0;
    }
    h8 mmB[2];
    uint32_t (*rows)[kDgStride] = nullptr;
    if constexpr (kMM) {
        mm_basis(L, mmB);
        rows = mm->dg[L.w];
        uint4 *z = reinterpret_cast<uint4 *>(&rows[L.l >> 3][(L.l & 7) * 8]);
        z[0] = make_uint4(0u, 0u, 0u, 0u);
        z[1] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (n == 0) return;            // no Gaussian, no gradient (uniform: every thread returns)
    BwdState st{1.f, 0.f, 0.f, 0.f, 0.f, 0};
    if (L.inside) {
        const int64_t p = int64_t(L.py) * v.W + int64_t(L.px);
        const int64_t HW = int64_t(v.H) * v.W;
        st.T = v.final_T[p];
        st.last = v.last_contrib[p];
        st.gr = v.dL_dimage[p]; st.gg = v.dL_dimage[HW + p]; st.gb = v.dL_dimage[2 * HW + p];
        st.beta = v.bg[0] * st.gr + v.bg[1] * st.gg + v.bg[2] * st.gb;   // (T_final (bg . g)) / T_final
    }
    __syncthreads();
    if (st.last > 0) atomicMax(&s_maxlast, st.last);
    __syncthreads();
    const uint2 rg = reinterpret_cast<const uint2 *>(v.ranges)[tile.y * v.gx + tile.x];
    const int64_t start = rg.x;
    // positions [0, max last) are the only ones that matter (never more than the list holds)
    // (the same value in every lane: made wavefront-uniform, so that the batch and group loops
    // and their index arithmetic run on the scalar unit)
    const int maxlast = __builtin_amdgcn_readfirstlane(s_maxlast);
    const int64_t len = maxlast < int64_t(rg.y) - int64_t(rg.x) ? maxlast
                                                                : int64_t(rg.y) - int64_t(rg.x);
    const int B = batch_bwd<NB>(len);
    const int nb = int((len + B - 1) / B);
    if (nb == 0) return;

    // List entries are loaded two batches ahead and attributes one batch ahead.
    const auto entry = [&](int bb) {          // batch bb's entry for this thread (bb may be < 0)
        const int64_t o = int64_t(bb) * B + L.t;
        return load_entry(plist, start + o, bb >= 0 && L.t < B && o < len, start);
    };
    // Each wavefront flushes a quarter of the batch's slots. It lists the slots that
    // received a nonzero sum, in slot order, and then spreads their nine sums over its lanes,
    // seven listed slots at a time: lane l < 63 adds sum l % 9 of slot l / 9, so that consecutive
    // lanes add consecutive words of one Gaussian (a wavefront's atomic instruction reaches about
    // 30 cache lines instead of 64), no lane is spent on the slots without a sum (over half of a
    // 3-sigma list's; six of a wavefront's 32 slots are listed on average on the 4K frame), and
    // the array and word that a lane adds to are the same for every slot: found once per tile, not
    // once per sum (4K BF16 backward 1% faster, 1080p 2%). Each
    // item is zeroed by the lane that reads it (an unlisted slot's sums are all +-0 already),
    // ready for batch bb - 1, which adds after the next barrier.
    // Deterministic form: the listed slots' rows are written by 16 lanes each, word k < 9 being the
    // four wavefronts' sum k of the slot added in wavefront order, and numbered among their
    // Gaussian's as they come (the gather puts them in order).
    const auto flush_det = [&](int bb, int filled) {
        const int per = (filled + 3) >> 2, s0 = L.w * per;
        uint16_t *list = det->list[L.w];
        uint32_t bits = 0u;
        if (L.l < per && s0 + L.l < filled) {
#pragma unroll
            for (int w = 0; w < kBlock / 64; ++w) {
                const float *p = det->v[w] + (s0 + L.l) * kGrad;
#pragma unroll
                for (int k = 0; k < kGrad; ++k) bits |= __float_as_uint(p[k]) & 0x7fffffffu;
            }
        }
        const bool touched = bits != 0u;
        const unsigned long long m = __ballot(touched);
        const int64_t first = start + int64_t(bb) * B;
        if (touched) {
            const uint32_t g = S.ids[s0 + L.l];
            const int64_t p = first + det->entry[s0 + L.l];
            if (g < n && p < v.det_pairs) v.det_seq[p] = atomicAdd(v.det_rows + g, 1u);
            list[__popcll(m & ((1ull << L.l) - 1ull))] = uint16_t(s0 + L.l);
        }
        __builtin_amdgcn_wave_barrier();
        const int listed = __popcll(m), k = L.l & 15;
#pragma unroll 1
        for (int i = L.l >> 4; i < listed; i += 4) {
            const int slot = list[i];
            const int64_t p = first + det->entry[slot];
            float sum = 0.f;
            if (k < kGrad) {
#pragma unroll
                for (int w = 0; w < kBlock / 64; ++w) {
                    float *q = det->v[w] + slot * kGrad + k;
                    sum += *q;
                    *q = 0.f;
                }
            }
            if (p < v.det_pairs) v.det_partial[p * kDetStride + k] = sum;
        }
        __builtin_amdgcn_wave_barrier();
    };
    constexpr int kItemSlots = 64 / kGrad;
    const int item_slot = L.l < kItemSlots * kGrad ? L.l / kGrad : NB, item_k = L.l % kGrad;
    if constexpr (!kDet) {
        if (L.t < 64)            // (ordered before the first flush by the batch loop's barrier)
            acc_->item[L.t] = {item_k < 3 ? v.dL_dconics + item_k
                               : item_k < 5 ? v.dL_dmeans2d + (item_k - 3)
                               : item_k == 5 ? v.dL_dopacity : v.dL_dcolors + (item_k - 6),
                               item_k < 3 ? 3u : item_k < 5 ? 2u : item_k == 5 ? 1u : 3u, 0u};
    }
    const auto flush = [&](int bb, int staged) {     // the sums of batch bb and its slots
        if constexpr (kDet) {
            flush_det(bb, staged);
            return;
        }
        BwdAcc<NB> &s_acc = *acc_;
        const int per = (staged + 3) >> 2;         // slots per wavefront, at most 64
        float *acc = s_acc.v;
        const uint32_t *ids = S.ids;
        uint16_t *list = s_acc.list[L.w];
        const int s0 = L.w * per;
        // a slot is listed if any of its nine sums is nonzero (NaN included); one whose sums
        // are all +-0 adds nothing to the gradients, whether or not a pair reached it
        bool touched = false;
        if (L.l < per && s0 + L.l < staged) {
            const float *p = acc + (s0 + L.l) * kGrad;
            uint32_t bits = 0u;
#pragma unroll
            for (int k = 0; k < kGrad; ++k) bits |= __float_as_uint(p[k]) & 0x7fffffffu;
            touched = bits != 0u;
        }
        const unsigned long long m = __ballot(touched);
        if (touched) list[__popcll(m & ((1ull << L.l) - 1ull))] = uint16_t(s0 + L.l);
        __builtin_amdgcn_wave_barrier();   // the list is written and read by this wavefront only
        const int listed = __popcll(m);
        const auto item = s_acc.item[L.l];
#pragma unroll 1
        for (int i = item_slot; i < listed; i += kItemSlots) {
            const int slot = list[i];
            float *p = acc + slot * kGrad + item_k;
            const float val = *p;
            *p = 0.f;
            if (val != 0.f) unsafeAtomicAdd(item.dst + size_t(ids[slot]) * item.stride, val);
        }
    };
    GRaw nxt = src.fetch(entry(nb - 1).id(), n);
    Entry ent = entry(nb - 2);
    if constexpr (kDet) {
        for (int e = L.t; e < NB * kGrad; e += kBlock) {
#pragma unroll
            for (int w = 0; w < kBlock / 64; ++w) det->v[w][e] = 0.f;
        }
    } else {
        for (int e = L.t; e < NB * kGrad; e += kBlock) acc_->v[e] = 0.f;
    }
    int staged = 0;                            // slots of the batch before
    for (int b = nb - 1; b >= 0; --b) {
        const int base = b * B;
        // as in the forward, only the entries that can reach the tile are staged, in order
        const Eval e = evaluate(nxt, xc, yc);
        uint32_t quad;
        const bool keep = keep_entry<M>(nxt, e, v.reach == 0, L.t < B && base + L.t < len, quad);
        const unsigned long long kept = __builtin_amdgcn_ballot_w64(keep);
        if (L.l == 0) S.kept[L.w] = kept;
        __syncthreads();             // every wavefront is done with batch b + 1
        // The batch's memory operations come before its compute, and the flush's atomics before the
        // loads of the next batch: the wait for those, a whole compute later, finds both done (with
        // the flush after the compute it would expose the atomics' latency).
        if (b + 1 < nb) flush(b + 1, staged);
        // entries kept before each wavefront's, and by this lane's wavefronts before a list position
        const uint4 ka = reinterpret_cast<const uint4 *>(S.kept)[0];
        const uint4 kb = reinterpret_cast<const uint4 *>(S.kept)[1];
        const int c0 = __popc(uniform(ka.x)) + __popc(uniform(ka.y));
        const int c1 = c0 + __popc(uniform(ka.z)) + __popc(uniform(ka.w));
        const int c2 = c1 + __popc(uniform(kb.x)) + __popc(uniform(kb.y));
        const int total = c2 + __popc(uniform(kb.z)) + __popc(uniform(kb.w));
        const auto before = [&](int w) { return w == 0 ? 0 : w == 1 ? c0 : w == 2 ? c1 : c2; };
        int slot = kNoSlot;
        if (keep) {
            slot = int(__builtin_amdgcn_mbcnt_hi(
                uint32_t(kept >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(kept), uint32_t(before(L.w)))));
            stage<M>(nxt, e, quad, slot, S);
            S.mean[slot] = make_float2(nxt.x, nxt.y);
        }
        const int ng = (total + kGroup - 1) / kGroup;
        if constexpr (M != Mode::Plain) {
            if (total + L.t < ng * kGroup) stage_inert<M>(total + L.t, S);
        }
        // slots below `last` hold entries up to the lane's last contributor
        int last;
        {
            const int r = st.last - base < B ? st.last - base : B;      // entries of this batch
            const int w = r > 0 ? (r - 1) >> 6 : 0, in = r - 64 * w;       // 1 <= in <= 64 if r > 0
            const unsigned long long m = S.kept[w];
            const unsigned long long low = in <= 0 ? 0ull : ~0ull >> (64 - in);
            last = before(w) + __popcll(m & low);
        }
        staged = total;
        __syncthreads();
        if (keep) {
            S.ids[slot] = nxt.id;
            if constexpr (kDet) det->entry[slot] = uint16_t(L.t);
        }
        // unconditional: before the first batch these read entry `start` and Gaussian 0, unused
        nxt = src.fetch(ent.id(), n);
        ent = entry(b - 2);
        for (int g = ng - 1; g >= 0; --g) {
            // nothing to do for this wave unless one of its pixels blended past the group's start
            // and (plain form) a Gaussian of the group can reach it
            if (__ballot(last > g * kGroup) == 0) continue;
            uint32_t reach = 0xffffu;
            if constexpr (M == Mode::Plain) {
                reach = group_reach(S, g * kGroup, total, L);
                if (reach == 0u) continue;
            }
            // the group's first slot, held in a vector register: each Gaussian's LDS addresses are
            // then immediate offsets from it (from a scalar base the compiler copies the base
            // into a vector register again for every Gaussian)
            int slot0 = g * kGroup;
            asm volatile("" : "+v"(slot0));
            const float4 *ga = &S.attr[slot0];   // the group's staged values
            const float2 *gb = &S.mean[slot0];
            // the group's sums, Gaussian 0 (deterministic: this wavefront's slice)
            float *accw = (kDet ? det->v[L.w] : acc_->v) + g * kGroup * kGrad;
            float *acc = accw + (kMM ? 0 : word);   // this lane's word (VALU reduction)
            const int rel = last - g * kGroup;      // slots < rel are in range
            // the whole group is in range for every lane (the common case once past the lanes'
            // last contributors; never for a partial tile, whose outside lanes have last = 0)
            const bool whole = __builtin_amdgcn_ballot_w64(rel < kGroup) == 0ull;
            f16x qm;
            if constexpr (M != Mode::Plain) qm = group_q<M, NB>(S, g * kGroup, L, bhi, blo);
            const auto q_of = [&](int u) {
                if constexpr (M == Mode::Plain) return plain_q(S.geo[slot0 + u], S.geo2[slot0 + u], L);
                else return qm[u];
            };
            if constexpr (kMM) {
                // two half-groups of 8: Gaussians 15..8, then 7..0, each followed by its product
#pragma unroll
                for (int h = 1; h >= 0; --h) {
                    unsigned hmask = 0u;
                    if (whole) {
#pragma unroll
                        for (int i = 7; i >= 0; --i) {
                            const int u = 8 * h + i;
                            if (((reach >> u) & 1u) == 0u) continue;
                            if (reverse_pair_mm<false>(q_of(u), true, ga, gb, u, L, st,
                                                       acc + u * kGrad, rows[i]))
                                hmask |= 1u << i;
                        }
                    } else {
#pragma unroll
                        for (int i = 7; i >= 0; --i) {
                            const int u = 8 * h + i;
                            if (((reach >> u) & 1u) == 0u) continue;
                            if (reverse_pair_mm<true>(q_of(u), u < rel, ga, gb, u, L, st,
                                                      acc + u * kGrad, rows[i]))
                                hmask |= 1u << i;
                        }
                    }
                    if (hmask != 0u)
                        mm_reduce(rows, mmB, hmask, gb + 8 * h, xc, yc, accw + 8 * h * kGrad, L);
                }
            } else if (whole) {
#pragma unroll
                for (int u = kGroup - 1; u >= 0; --u) {
                    if (((reach >> u) & 1u) == 0u) continue;
                    reverse_pair<false>(q_of(u), true, ga, gb, u, L, st, acc + u * kGrad);
                }
            } else {
#pragma unroll
                for (int u = kGroup - 1; u >= 0; --u) {
                    if (((reach >> u) & 1u) == 0u) continue;
                    reverse_pair<true>(q_of(u), u < rel, ga, gb, u, L, st, acc + u * kGrad);
                }
            }
        }
    }
    __syncthreads();
    flush(0, staged);
}

// ------------------------------------------------------------------------------- kernels
// Wavefronts per SIMD that a kernel's launch bound asks for: its register target, but never more
// than the blocks that fit in a compute unit's 160 KB of LDS (a 256-thread block puts one
// wavefront on each SIMD), so the compiler is not held to an occupancy the LDS rules out.
constexpr size_t kLdsPerCu = 160 * 1024;
constexpr int fit_waves(int target, size_t lds) {
    return int(kLdsPerCu / lds) < target ? int(kLdsPerCu / lds) : target;
}
// LDS of one block: the staged batches (and, backward, the gradient accumulators), plus the few
// scalars the kernels share
template <Mode M, int NB> constexpr size_t lds_fwd() { return sizeof(FwdStage<M, NB>) + 64; }
template <Mode M, int NB, bool kMM> constexpr size_t lds_bwd() {
    return sizeof(BwdStage<M, NB>) + sizeof(BwdAcc<NB>) + (kMM ? sizeof(BwdMM) : 0) + 64;
}
// The transposition tiles exist only in the matrix-core reduction's kernels.
struct NoMM {};
template <bool kMM> using MMTiles = typename std::conditional<kMM, BwdMM, NoMM>::type;
template <bool kMM> __device__ inline BwdMM *mm_ptr(MMTiles<kMM> &t) {
    if constexpr (kMM) return &t;
    else return nullptr;
}
// Register targets of the one-tile-per-block backward kernels; the matrix-core reduction keeps
// the product's operands and results live across each half-group and needs more registers
// (fewer targets spill). (6 wavefronts per SIMD for the GEMM forms fit in LDS, 26.9 KB per block,
// but at 80 registers a few values spill and the backward is about 1% slower than at 5.)
template <Mode M, bool kMM> constexpr int waves_bwd_tile() {
    return kMM ? (M == Mode::Plain ? 5 : 4) : (M == Mode::Plain ? 7 : 5);
}
// Forward: small grids, all of whose blocks are on the GPU at once also with the registers for a group
// read ahead, are bound by each wavefront's own chain (an LDS read after a branch for each Gaussian),
// not by instruction issue. Read ahead, FP16: 256 tiles 35 -> 29 us, 512 tiles 35 -> 31, 1024 tiles
// 40 -> 37.5; 1536 tiles, past the rule, 47 -> 55. FP32, which holds its geometry too and has half
// the blocks: 512 tiles 47 -> 41, 768 tiles 49 -> 67. (The backward gains 1%: its chain is the
// reduction.)
template <Mode M, bool kFew> constexpr int waves_fwd_tile() {
    return kFew ? (M == Mode::Plain ? 2 : 4) : (M == Mode::Plain ? 8 : 7);
}
constexpr int kCus = 256;
template <Mode M> inline bool few_tiles(int64_t n_tiles) {
    return n_tiles <= kCus * waves_fwd_tile<M, true>();
}
__device__ inline TileXY view_tile(const ViewDesc &v, uint32_t rank) {
    return strip_tile(rank, uint32_t(v.gx), uint32_t(v.H + kTile - 1) / kTile);
}
// Single view: block b renders the tile of rank xcd_rank(b).
template <Mode M, int NB, bool kFew = false, bool kAll = false>
__global__ __launch_bounds__(kBlock, fit_waves(waves_fwd_tile<M, kFew>(), lds_fwd<M, NB>()))
void k_blend_fwd(ViewDesc v) {
    __shared__ FwdStage<M, NB> S[kFwdBuffers<kAll>];
    const uint32_t rank = xcd_rank(blockIdx.x, uint32_t(v.n_tiles));
    if (rank >= uint32_t(v.n_tiles)) return;
    const TileXY tile = view_tile(v, rank);
    fwd_tile<M, NB, false, kFew, kAll>(v, tile, S);
}

template <Mode M, int NB, bool kMM>
__global__ __launch_bounds__(kBlock, fit_waves(waves_bwd_tile<M, kMM>(), lds_bwd<M, NB, kMM>()))
void k_blend_bwd(ViewDesc v) {
    __shared__ BwdStage<M, NB> S;
    __shared__ BwdAcc<NB> s_acc;   // per-Gaussian gradient sums of the current batch
    __shared__ MMTiles<kMM> s_mm;
    __shared__ int s_maxlast;
    const uint32_t rank = xcd_rank(blockIdx.x, uint32_t(v.n_tiles));
    if (rank >= uint32_t(v.n_tiles)) return;
    const TileXY tile = view_tile(v, rank);
    bwd_tile<M, NB, kMM>(v, tile, S, &s_acc, s_maxlast, mm_ptr<kMM>(s_mm));
}

// Single view, packed records (gsb_pack_gaussians): the default launch shape (LDS batches of 256,
// vector-ALU reduction), attributes from one 48-byte record per list entry.
template <Mode M, bool kFew, bool kAll>
__global__ __launch_bounds__(kBlock, fit_waves(waves_fwd_tile<M, kFew>(), lds_fwd<M, kDefaultBatchFwd>()))
void k_blend_fwd_rec(ViewDesc v) {
    constexpr int NB = kAll ? kAllBatchFwd : kDefaultBatchFwd;
    __shared__ FwdStage<M, NB> S[kFwdBuffers<kAll>];
    const uint32_t rank = xcd_rank(blockIdx.x, uint32_t(v.n_tiles));
    if (rank >= uint32_t(v.n_tiles)) return;
    const TileXY tile = view_tile(v, rank);
    fwd_tile<M, NB, true, kFew, kAll>(v, tile, S);
}

template <Mode M>
__global__ __launch_bounds__(kBlock, fit_waves(waves_bwd_tile<M, false>(), lds_bwd<M, kDefaultBatchBwd, false>()))
void k_blend_bwd_rec(ViewDesc v) {
    __shared__ BwdStage<M, kDefaultBatchBwd> S;
    __shared__ BwdAcc<kDefaultBatchBwd> s_acc;
    __shared__ int s_maxlast;
    const uint32_t rank = xcd_rank(blockIdx.x, uint32_t(v.n_tiles));
    if (rank >= uint32_t(v.n_tiles)) return;
    const TileXY tile = view_tile(v, rank);
    bwd_tile<M, kDefaultBatchBwd, false, true>(v, tile, S, &s_acc, s_maxlast, nullptr);
}

// Deterministic backward, one tile per block: LDS for batches of 128 (the four wavefront slices of the
// batch sums take four times the LDS of the shared accumulator), lists of up to 256 entries in batches
// of 64 (batch_bwd); records as attributes.
constexpr int kDetBatch = 128;
template <Mode M> constexpr size_t lds_bwd_det() {
    return sizeof(BwdStage<M, kDetBatch>) + sizeof(BwdAccDet<kDetBatch>) + 64;
}
template <Mode M>
__global__ __launch_bounds__(kBlock, fit_waves(waves_bwd_tile<M, false>(), lds_bwd_det<M>()))
void k_blend_bwd_det(ViewDesc v) {
    __shared__ BwdStage<M, kDetBatch> S;
    __shared__ BwdAccDet<kDetBatch> s_det;
    __shared__ int s_maxlast;
    const uint32_t rank = xcd_rank(blockIdx.x, uint32_t(v.n_tiles));
    if (rank >= uint32_t(v.n_tiles)) return;
    const TileXY tile = view_tile(v, rank);
    bwd_tile<M, kDetBatch, false, true, true>(v, tile, S, nullptr, s_maxlast, nullptr, &s_det);
}

// Gaussians with more than kDetWaveRows rows are listed (word 0: how many) for blocks of their own; those
// of up to kDetCountRows rows are put in order by counting there, others by a sort.
constexpr uint32_t kDetWaveRows = 64, kDetCountRows = 256;
// No rows yet: counts per Gaussian, numbers per list position.
__global__ __launch_bounds__(256) void k_det_init(uint32_t *rows, int64_t n, uint32_t *seq,
                                                  int64_t pairs, uint32_t *large) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) rows[i] = 0u;
    if (i < pairs) seq[i] = ~0u;
    if (i == 0) large[0] = 0u;
}

// The positions with a row, by Gaussian (first: the scanned counts). Against a stable sort of all
// list positions by Gaussian (three passes, each with its counts and scan: 103 us for 150 k Gaussians
// at 997 x 613) this leaves the order within a Gaussian to the gather: 27 us with the counts' scan.
// (Ranges that overlap could count more rows than there are positions: those are left out.)
__global__ __launch_bounds__(256) void k_det_place(const uint32_t *plist, const uint32_t *seq,
                                                   int64_t pairs, const uint32_t *first, int64_t n,
                                                   uint32_t *list, uint32_t *large) {
    const int64_t i0 = int64_t(blockIdx.x) * 1024 + threadIdx.x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t i = i0 + 256 * k;
        if (i >= pairs) continue;
        const uint32_t nth = seq[i], g = plist[i];
        if (nth == ~0u || g >= uint64_t(n)) continue;
        const uint64_t at = uint64_t(first[g]) + nth;
        if (at < uint64_t(pairs)) list[at] = uint32_t(i);
        if (nth == kDetWaveRows) {               // one of each such Gaussian's
            const uint32_t o = atomicAdd(large, 1u);
            if (o < uint64_t(pairs) / kDetWaveRows) large[1 + o] = g;
        }
    }
}

// More than kDetCountRows rows: list[0, m) in increasing order, by a stable radix sort between `list` and
// `other` of the block's four wavefronts, kDetBits of the positions' range a pass; returns which of the
// two holds it. A wavefront counts and places a quarter of the list, 64 at a time, so that the steps
// grow with m alone. (One wavefront that counted the rows per tile, 1024 tiles at a time, read the
// list and the rows again for every 1024 tiles: the gather of 16 Gaussians that are on each of the
// 32400 tiles of a 4K frame took 84.1 ms, now 0.29; of 8 with 600 px at 1080p 2.54 ms, now 0.08.)
constexpr int kDetBits = 9, kDetRadix = 1 << kDetBits;
__device__ inline const uint32_t *det_order(uint32_t *list, uint32_t *other, uint32_t m,
                                            uint32_t (*cnt)[kDetRadix], uint32_t *s_red, int w, int lane) {
    constexpr int kWaves = 4, kAhead = 4, kOwn = kDetRadix / (64 * kWaves);
    const uint32_t seg = (m + 64 * kWaves - 1) / (64 * kWaves) * 64;
    const uint32_t j0 = uint32_t(w) * seg, j1 = j0 + seg < m ? j0 + seg : m;
    // f(key, whether there is one) for this wavefront's part, in order, kAhead loads at a time
    const auto each = [&](const uint32_t *from, auto f) {
        for (uint32_t j = j0; j < j1; j += 64 * kAhead) {                     // uniform
            uint32_t k[kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const uint32_t i = j + 64 * q + lane;
                k[q] = from[i < j1 ? i : j1 - 1];
            }
#pragma unroll
            for (int q = 0; q < kAhead; ++q) f(k[q], j + 64 * q + lane < j1);
        }
    };
    uint32_t lo = ~0u, hi = 0u;
    each(list, [&](uint32_t k, bool) {
        lo = k < lo ? k : lo;
        hi = k > hi ? k : hi;
    });
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const uint32_t a = __shfl_xor(lo, o, 64), b = __shfl_xor(hi, o, 64);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    if (lane == 0) {
        s_red[w] = lo;
        s_red[kWaves + w] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
        lo = s_red[i] < lo ? s_red[i] : lo;
        hi = s_red[kWaves + i] > hi ? s_red[kWaves + i] : hi;
    }
    __syncthreads();
    lo = uint32_t(__builtin_amdgcn_readfirstlane(int(lo)));
    hi = uint32_t(__builtin_amdgcn_readfirstlane(int(hi)));
    const int t = 64 * w + lane;
    for (int shift = 0; shift < 32 && ((hi - lo) >> shift) != 0u; shift += kDetBits) {     // uniform
        const auto digit = [&](uint32_t k) { return ((k - lo) >> shift) & uint32_t(kDetRadix - 1); };
        for (int d = lane; d < kDetRadix; d += 64) cnt[w][d] = 0u;
        __builtin_amdgcn_wave_barrier();
        each(list, [&](uint32_t k, bool valid) {
            if (valid) atomicAdd(&cnt[w][digit(k)], 1u);
        });
        __syncthreads();
        // where each wavefront's positions of a digit start: digits before, then wavefronts before
        uint32_t sum = 0;
#pragma unroll
        for (int q = 0; q < kOwn; ++q) {
#pragma unroll
            for (int i = 0; i < kWaves; ++i) sum += cnt[i][t * kOwn + q];
        }
        uint32_t x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        uint32_t run = x - sum;
        if (lane == 63) s_red[w] = x;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kWaves; ++i) run += i < w ? s_red[i] : 0u;
#pragma unroll
        for (int q = 0; q < kOwn; ++q) {
#pragma unroll
            for (int i = 0; i < kWaves; ++i) {
                const uint32_t c = cnt[i][t * kOwn + q];
                cnt[i][t * kOwn + q] = run;
                run += c;
            }
        }
        __syncthreads();
        each(list, [&](uint32_t k, bool valid) {
            const uint32_t d = digit(k);
            unsigned long long same = __builtin_amdgcn_ballot_w64(valid);      // lanes with this digit
#pragma unroll
            for (int b = 0; b < kDetBits; ++b) {
                const bool set = ((d >> b) & 1u) != 0u;
                const unsigned long long vote = __builtin_amdgcn_ballot_w64(set);
                same &= set ? vote : ~vote;
            }
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
                uint32_t(same >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(same), 0u));
            if (valid) {
                const uint32_t at = cnt[w][d];
                if (rank == 0u) cnt[w][d] = at + uint32_t(__popcll(same));
                other[at + rank] = k;
            }
        });
        __syncthreads();
        uint32_t *swap = list;
        list = other;
        other = swap;
    }
    return list;
}

// list[0, m), m <= kDetCountRows, into increasing order in s_key: each thread of the block counts the
// positions before its own. (By a wavefront for its four Gaussians, one after the other, the whole call for
// 25 Gaussians on each of 208 tiles took 92 us, now 49, and the gather of 2000 of up to some 400 rows
// at 4K 84, now 58.)
__device__ inline void det_count_order(const uint32_t *list, uint32_t m, uint32_t *s_key) {
    const uint32_t t = threadIdx.x;
    const uint32_t key = t < m ? list[t] : ~0u;
    s_key[t] = key;
    __syncthreads();
    uint32_t at = 0;
    for (uint32_t j = 0; j < m; j += 4) {
        const uint4 k = *reinterpret_cast<const uint4 *>(s_key + j);
        at += (k.x < key ? 1u : 0u) + (k.y < key ? 1u : 0u) + (k.z < key ? 1u : 0u) + (k.w < key ? 1u : 0u);
    }
    __syncthreads();
    if (t < m) s_key[at] = key;
    __syncthreads();
}

// The gradients of Gaussian g from its nine sums, as k_bwd_finish forms them.
struct DetOut {
    const float4 *rec;
    float *dmeans, *dconics, *dopac, *dcolors;
};
__device__ inline void det_store(const DetOut &out, int64_t g, const float *t) {
    const float4 r0 = out.rec[3 * g], r1 = out.rec[3 * g + 1];
    const float A = r0.z, B = r0.w, C = r1.x;
    out.dconics[3 * g] = -0.5f * t[0];
    out.dconics[3 * g + 1] = -t[1];
    out.dconics[3 * g + 2] = -0.5f * t[2];
    out.dmeans[2 * g] = -(A * t[3] + B * t[4]);
    out.dmeans[2 * g + 1] = -(B * t[3] + C * t[4]);
    out.dopac[g] = opacity_grad(t[5], r1.y);
    out.dcolors[3 * g] = t[6];
    out.dcolors[3 * g + 1] = t[7];
    out.dcolors[3 * g + 2] = t[8];
}

// How many of the 16 lanes' keys are less than this lane's.
template <int kRor>
__device__ inline uint32_t row_rank(uint32_t key) {
    if constexpr (kRor == 16) {
        return 0u;
    } else {
        const uint32_t o = uint32_t(__builtin_amdgcn_update_dpp(0, int(key), 0x120 + kRor, 0xf, 0xf, true));
        return (o < key ? 1u : 0u) + row_rank<kRor + 1>(key);
    }
}

// Per Gaussian: its rows' sums in the order of the list positions, in a fixed reduction tree. Four
// Gaussians per wavefront, 16 lanes each, where they have up to 16 rows (most do): the positions are
// ranked within the 16 lanes, lane j adds the row of rank j. Those with more take the whole wavefront
// in turn, up to 64. (A wavefront for each Gaussian took 51 us of 150 k Gaussians, this 27; a thread for
// each would leave most lanes idle behind the largest footprint.)
// The listed ones, with more than kDetWaveRows, are the first kDetBlocks blocks' (four per compute unit;
// they cost nothing measurable where there are none), a block at a time each. Up to kDetCountRows its
// first wavefront adds the rows of rank l, l + 64, ... in lane l, beyond that thread t those of rank t,
// t + 256, ..., and the four wavefronts' sums are added in order.
constexpr int kGatherPer = 4, kDetBlocks = 1024;
__global__ __launch_bounds__(256, 7) void k_det_gather(DetOut out, const float *partial,
                                                    const uint32_t *first, const uint32_t *rows,
                                                    uint32_t *list, uint32_t *other,
                                                    const uint32_t *large, int64_t pairs, int64_t n) {
    static_assert(kDetCountRows <= 256 && kDetCountRows <= kDetRadix, "a thread and a word for each position");
    __shared__ __align__(16) uint32_t s_cnt[4][kDetRadix];
    __shared__ uint32_t s_red[8];
    __shared__ float s_sum[4][kGrad];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, j = lane & 15;
    // the rows of Gaussian g in the list: from place a, m of them
    const auto rows_of = [&](int64_t g, uint32_t &a) {
        a = first[g];
        const int64_t room = pairs - int64_t(a), have = rows[g];
        return uint32_t(have < room ? have : room > 0 ? room : 0);
    };
    float sum[kGrad];
    const auto clear = [&] {
#pragma unroll
        for (int k = 0; k < kGrad; ++k) sum[k] = 0.f;
    };
    const auto add = [&](uint32_t pos) {
        if (pos >= uint64_t(pairs)) return;
        const float *p = partial + int64_t(pos) * kDetStride;
        const float4 p0 = *reinterpret_cast<const float4 *>(p);
        const float4 p1 = *reinterpret_cast<const float4 *>(p + 4);
        sum[0] += p0.x; sum[1] += p0.y; sum[2] += p0.z; sum[3] += p0.w;
        sum[4] += p1.x; sum[5] += p1.y; sum[6] += p1.z; sum[7] += p1.w;
        sum[8] += p[8];
    };
    // the wavefront's nine sums, in every lane
    const auto total = [&](float (&t)[kGrad]) {
        float ab, c;
        wave_sum9(sum, lane, ab, c);
        // lane 16r holds sum {0,2,1,3}[r], lane 16r + 8 sum 4 + {0,2,1,3}[r]; lane 0 of c sum 8
        const auto from = [](float x, int l) {
            return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
        };
        t[0] = from(ab, 0);  t[2] = from(ab, 16); t[1] = from(ab, 32); t[3] = from(ab, 48);
        t[4] = from(ab, 8);  t[6] = from(ab, 24); t[5] = from(ab, 40); t[7] = from(ab, 56);
        t[8] = from(c, 0);
    };
    if (blockIdx.x < kDetBlocks) {               // block-uniform
        const uint64_t room = uint64_t(pairs) / kDetWaveRows, have = large[0];
        for (uint64_t b = blockIdx.x; b < (have < room ? have : room); b += kDetBlocks) {
            const uint32_t g = large[1 + b];
            uint32_t a = 0u;
            const uint32_t m = g < n ? rows_of(g, a) : 0u;
            if (m <= kDetWaveRows) continue;     // block-uniform
            if (m <= kDetCountRows) {
                det_count_order(list + a, m, s_cnt[0]);
                if (w == 0) {
                    clear();
                    for (uint32_t k = lane; k < m; k += 64) add(s_cnt[0][k]);
                    float t[kGrad];
                    total(t);
                    if (lane == 0) det_store(out, g, t);
                }
                __syncthreads();                 // (before the next one's are written there)
                continue;
            }
            const uint32_t *order = det_order(list + a, other + a, m, s_cnt, s_red, w, lane);
            clear();
            for (uint32_t k = threadIdx.x; k < m; k += 4 * 256) {
                uint32_t p[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) p[q] = k + 256 * q < m ? order[k + 256 * q] : ~0u;
#pragma unroll
                for (int q = 0; q < 4; ++q) add(p[q]);       // (~0: no row)
            }
            float t[kGrad];
            total(t);
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < kGrad; ++k) s_sum[w][k] = t[k];
            }
            __syncthreads();
            if (threadIdx.x == 0) {
#pragma unroll
                for (int k = 0; k < kGrad; ++k)
                    t[k] = ((s_sum[0][k] + s_sum[1][k]) + s_sum[2][k]) + s_sum[3][k];
                det_store(out, g, t);
            }
            __syncthreads();
        }
        return;
    }
    const int64_t wave = ((int64_t(blockIdx.x) - kDetBlocks) * blockDim.x + threadIdx.x) >> 6;
    const int64_t g0 = wave * kGatherPer, g = g0 + (lane >> 4);
    uint32_t a = 0u, m = 0u;
    if (g < n) m = rows_of(g, a);
    clear();
    const bool mine = m <= 16u && uint32_t(j) < m;
    const uint32_t key = mine ? list[a + uint32_t(j)] : ~0u;
    const uint32_t rank = row_rank<1>(key);
    const uint32_t pos = uint32_t(__builtin_amdgcn_ds_permute(
        4 * ((lane & 48) + (mine ? int(rank) : j)), int(key)));
    if (mine) add(pos);
#pragma unroll
    for (int k = 0; k < kGrad; ++k) {
        float x = sum[k];
        x = dpp_add2<0x128>(x, x);               // rotations within the 16 lanes by 8, 4, 2, 1
        x = dpp_add2<0x124>(x, x);
        x = dpp_add2<0x122>(x, x);
        sum[k] = dpp_add2<0x121>(x, x);
    }
    if (g < n && m <= 16u && j == 0) det_store(out, g, sum);
#pragma unroll 1
    for (int r = 0; r < kGatherPer; ++r) {
        const uint32_t mr = uint32_t(__builtin_amdgcn_readlane(int(m), 16 * r));
        if (mr <= 16u || mr > kDetWaveRows) continue;        // uniform (m is 0 past the last Gaussian)
        const uint32_t ar = uint32_t(__builtin_amdgcn_readlane(int(a), 16 * r));
        clear();
        const bool has = uint32_t(lane) < mr;
        const uint32_t k64 = has ? list[ar + uint32_t(lane)] : ~0u;
        int at = 0;
        for (int k = 0; k < int(mr); ++k)
            at += uint32_t(__builtin_amdgcn_readlane(int(k64), k)) < k64 ? 1 : 0;
        const uint32_t p = uint32_t(__builtin_amdgcn_ds_permute(4 * (has ? at : lane), int(k64)));
        if (has) add(p);
        float t[kGrad];
        total(t);
        if (lane == 0) det_store(out, g0 + r, t);
    }
}

// One record per Gaussian: (x, y, A, B), (C, o, r, g), (b, 0, 0, 0). A block assembles its 256
// records in LDS and writes them out as consecutive 16-byte words, so that every store
// instruction covers one contiguous kilobyte (thread t writing its own record's three words at a
// 48-byte stride wrote 18% more bytes than the records hold).
__global__ __launch_bounds__(256) void k_pack(const float2 *means, const F3 *conics,
                                              const float *opac, const F3 *colors, int64_t n,
                                              float4 *rec) {
    __shared__ float4 s_rec[3 * 256];
    const int t = threadIdx.x;
    const int64_t i0 = int64_t(blockIdx.x) * 256;
    const int64_t i = i0 + t;
    if (i < n) {
        const float2 m = means[i];
        const F3 c = conics[i], col = colors[i];
        s_rec[3 * t] = make_float4(m.x, m.y, c.a, c.b);
        s_rec[3 * t + 1] = make_float4(c.c, opac[i], col.a, col.b);
        s_rec[3 * t + 2] = make_float4(col.c, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    const int words = 3 * int(n - i0 < 256 ? n - i0 : 256);   // the block has at least one record
    for (int k = t; k < words; k += 256) rec[3 * i0 + k] = s_rec[k];
}

// Many views, one persistent launch. The (view, tile) items are split into 8 queues, one per XCD:
// queue x holds the ranks [n_tiles * x / 8, n_tiles * (x + 1) / 8) of every view (tiles in the
// strip order of strip_tile), views in plan
// order (heaviest per-tile cost first). A block serves the queue of its own XCD (block b runs on
// XCD b % 8) so that neighbouring tiles share that XCD's L2, and moves on to the next queue when
// its own is empty, so every block exits once all queues are drained.
// prefix[x * (n_views + 1) + k] = items of queue x that belong to views before k.
struct Queues {
    const ViewDesc *views;
    const int64_t *prefix;
    unsigned int *counters;    // 8 per direction
    int n_views;
};

__device__ inline int64_t band_lo(int64_t n_tiles, int x) { return n_tiles * x / kXcds; }

// The descriptor of a (block-uniform) view, read through the constant address space: no kernel
// writes the table, and only so does the compiler read it with scalar loads into scalar registers
// also inside the persistent loop, whose stores might alias it otherwise.
__device__ inline ViewDesc load_view(const Queues &Q, int view) {
    typedef const __attribute__((address_space(4))) uint32_t *ConstWords;
    static_assert(sizeof(ViewDesc) % 4 == 0, "copied by words");
    constexpr int kWords = int(sizeof(ViewDesc) / 4);
    const ConstWords src = (ConstWords)(reinterpret_cast<const uint32_t *>(Q.views + view));
    uint32_t w[kWords];
#pragma unroll
    for (int k = 0; k < kWords; ++k) w[k] = src[k];
    ViewDesc vd;
    __builtin_memcpy(&vd, w, sizeof(vd));
    return vd;
}

// The thread's index, opaque to the compiler in each iteration of the persistent loop: what a tile
// derives from it (pixel coordinates, bases, masks) is formed again per tile instead of being kept
// in registers across the loop.
__device__ inline int loop_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Next item for the calling block (thread 0 only): returns false when every queue is drained.
__device__ inline bool next_item(const Queues &Q, int &q, int &tried, int &view, uint32_t &rank) {
    while (tried < kXcds) {
        const int64_t *pre = Q.prefix + int64_t(q) * (Q.n_views + 1);
        const int64_t total = pre[Q.n_views];
        const int64_t i = total > 0 ? int64_t(atomicAdd(&Q.counters[q], 1u)) : total;
        if (i < total) {
            int lo = 0, hi = Q.n_views - 1;       // last k with pre[k] <= i
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (pre[mid] <= i) lo = mid; else hi = mid - 1;
            }
            view = lo;
            rank = uint32_t(band_lo(Q.views[lo].n_tiles, q) + (i - pre[lo]));
            return true;
        }
        q = (q + 1) % kXcds;
        ++tried;
    }
    return false;
}

// Register budgets for the persistent kernels (waves per SIMD): left alone the compiler spreads
// their registers over the loop and gives up a wave or more against the single-view kernels;
// these are the highest targets reached without spilling.
template <Mode M> constexpr int waves_fwd() { return M == Mode::Plain ? 8 : 7; }
template <Mode M> constexpr int waves_bwd() { return M == Mode::Plain ? 6 : 5; }

template <Mode M, int NB, bool kAll = false>
__global__ __launch_bounds__(kBlock, fit_waves(waves_fwd<M>(), lds_fwd<M, NB>()))
void k_blend_fwd_batched(Queues Q) {
    __shared__ FwdStage<M, NB> S[kFwdBuffers<kAll>];
    __shared__ int s_view;
    __shared__ uint32_t s_rank;
    int q = int(blockIdx.x % kXcds), tried = 0;
    for (;;) {
        if (threadIdx.x == 0) {
            int view = -1;
            uint32_t rank = 0;
            if (!next_item(Q, q, tried, view, rank)) view = -1;
            s_view = view;
            s_rank = rank;
        }
        __syncthreads();
        // the item is block-uniform: move it to scalar registers so the view descriptor is read
        // with scalar loads and its pointers stay in SGPRs
        const int view = __builtin_amdgcn_readfirstlane(s_view);
        const uint32_t rank = __builtin_amdgcn_readfirstlane(s_rank);
        __syncthreads();
        if (view < 0) break;
        const ViewDesc vd = load_view(Q, view);
        fwd_tile<M, NB, false, false, kAll>(vd, view_tile(vd, rank), S, loop_tid());
        __syncthreads();
    }
}

template <Mode M, int NB, bool kMM>
__global__ __launch_bounds__(kBlock, fit_waves(kMM ? 3 : waves_bwd<M>(), lds_bwd<M, NB, kMM>()))
void k_blend_bwd_batched(Queues Q) {
    __shared__ BwdStage<M, NB> S;
    __shared__ BwdAcc<NB> s_acc;
    __shared__ MMTiles<kMM> s_mm;
    __shared__ int s_maxlast;
    __shared__ int s_view;
    __shared__ uint32_t s_rank;
    int q = int(blockIdx.x % kXcds), tried = 0;
    for (;;) {
        if (threadIdx.x == 0) {
            int view = -1;
            uint32_t rank = 0;
            if (!next_item(Q, q, tried, view, rank)) view = -1;
            s_view = view;
            s_rank = rank;
        }
        __syncthreads();
        const int view = __builtin_amdgcn_readfirstlane(s_view);
        const uint32_t rank = __builtin_amdgcn_readfirstlane(s_rank);
        __syncthreads();
        if (view < 0) break;
        const ViewDesc vd = load_view(Q, view);
        bwd_tile<M, NB, kMM>(vd, view_tile(vd, rank), S, &s_acc, s_maxlast,
                             mm_ptr<kMM>(s_mm), nullptr, loop_tid());
        __syncthreads();
    }
}

// The same items in one non-persistent launch: block b takes item b / 8 of queue b % 8 (the
// dispatcher places block b on XCD b % 8 and hands out blocks in index order, so each XCD still
// walks its own bands heaviest view first). No loop state: registers as in the single-view
// kernels.
__device__ inline bool grid_item(const Queues &Q, int64_t b, int &view, uint32_t &rank) {
    const int x = int(b % kXcds);
    const int64_t i = b / kXcds;
    const int64_t *pre = Q.prefix + int64_t(x) * (Q.n_views + 1);
    if (i >= pre[Q.n_views]) return false;
    int lo = 0, hi = Q.n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= i) lo = mid; else hi = mid - 1;
    }
    view = lo;
    rank = uint32_t(band_lo(Q.views[lo].n_tiles, x) + (i - pre[lo]));
    return true;
}

template <Mode M, int NB, bool kAll = false>
__global__ __launch_bounds__(kBlock, fit_waves(M == Mode::Plain ? 8 : 7, lds_fwd<M, NB>()))
void k_blend_fwd_grid(Queues Q) {
    __shared__ FwdStage<M, NB> S[kFwdBuffers<kAll>];
    int view;
    uint32_t rank;
    if (!grid_item(Q, blockIdx.x, view, rank)) return;
    const ViewDesc vd = load_view(Q, view);
    fwd_tile<M, NB, false, false, kAll>(vd, view_tile(vd, rank), S);
}

template <Mode M, int NB, bool kMM>
__global__ __launch_bounds__(kBlock, fit_waves(waves_bwd_tile<M, kMM>(), lds_bwd<M, NB, kMM>()))
void k_blend_bwd_grid(Queues Q) {
    __shared__ BwdStage<M, NB> S;
    __shared__ BwdAcc<NB> s_acc;
    __shared__ MMTiles<kMM> s_mm;
    __shared__ int s_maxlast;
    int view;
    uint32_t rank;
    if (!grid_item(Q, blockIdx.x, view, rank)) return;
    const ViewDesc vd = load_view(Q, view);
    bwd_tile<M, NB, kMM>(vd, view_tile(vd, rank), S, &s_acc, s_maxlast, mm_ptr<kMM>(s_mm));
}

// Raw sums -> gradients of the stored scalars: d/dA = -S_xx/2, d/dB = -S_xy, d/dC = -S_yy/2,
// d/dx = -(A S_x + B S_y), d/dy = -(B S_x + C S_y) (power = -A dx^2/2 - B dx dy - C dy^2/2).
// blockIdx.y selects the view.
__global__ __launch_bounds__(256) void k_bwd_finish(const ViewDesc *views, ViewDesc single) {
    const ViewDesc &v = views ? views[blockIdx.y] : single;
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= v.n) return;
    F3 c;
    float o;
    if (v.records) {                 // (x, y, A, B), (C, o, ...): conic and opacity from the record
        const float4 r0 = v.records[3 * i], r1 = v.records[3 * i + 1];
        c = F3{r0.z, r0.w, r1.x};
        o = r1.y;
    } else {
        c = reinterpret_cast<const F3 *>(v.conics)[i];
        o = v.opacity[i];
    }
    v.dL_dopacity[i] = opacity_grad(v.dL_dopacity[i], o);
    F3 *dc = reinterpret_cast<F3 *>(v.dL_dconics);
    float2 *dm = reinterpret_cast<float2 *>(v.dL_dmeans2d);
    const F3 s = dc[i];
    const float2 m = dm[i];
    dc[i] = F3{-0.5f * s.a, -s.b, -0.5f * s.c};
    dm[i] = make_float2(-(c.a * m.x + c.b * m.y), -(c.b * m.x + c.c * m.y));
}

// Zero every gradient output (graph-capturable: a kernel, not a memset). blockIdx.y = view.
__global__ __launch_bounds__(256) void k_zero_grads(const ViewDesc *views, ViewDesc single) {
    const ViewDesc &v = views ? views[blockIdx.y] : single;
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= v.n) return;
    v.dL_dmeans2d[2 * i] = 0.f; v.dL_dmeans2d[2 * i + 1] = 0.f;
    v.dL_dconics[3 * i] = 0.f; v.dL_dconics[3 * i + 1] = 0.f; v.dL_dconics[3 * i + 2] = 0.f;
    v.dL_dopacity[i] = 0.f;
    v.dL_dcolors[3 * i] = 0.f; v.dL_dcolors[3 * i + 1] = 0.f; v.dL_dcolors[3 * i + 2] = 0.f;
}

__global__ void k_reset_counters(unsigned int *c, int m) {
    if (int(threadIdx.x) < m) c[threadIdx.x] = 0u;
}

// ------------------------------------------------------------------------------- dispatch
bool valid_batch(int nb) { return nb == 64 || nb == 128 || nb == 256; }

template <Mode M>
void launch_fwd_single(const ViewDesc &v, int nb, hipStream_t s) {
    const dim3 grid(unsigned(xcd_grid(v.n_tiles)));
    if (nb == 64) k_blend_fwd<M, 64><<<grid, kBlock, 0, s>>>(v);
    else if (nb == 128) k_blend_fwd<M, 128><<<grid, kBlock, 0, s>>>(v);
    else if (few_tiles<M>(v.n_tiles))
        (v.reach ? k_blend_fwd<M, 256, true> : k_blend_fwd<M, kAllBatchFwd, true, true>)<<<grid, kBlock, 0, s>>>(v);
    else
        (v.reach ? k_blend_fwd<M, 256> : k_blend_fwd<M, kAllBatchFwd, false, true>)<<<grid, kBlock, 0, s>>>(v);
}

template <Mode M, bool kMM>
void launch_bwd_single(const ViewDesc &v, int nb, hipStream_t s) {
    const dim3 grid(unsigned(xcd_grid(v.n_tiles)));
    if (nb == 64) k_blend_bwd<M, 64, kMM><<<grid, kBlock, 0, s>>>(v);
    else if (nb == 128) k_blend_bwd<M, 128, kMM><<<grid, kBlock, 0, s>>>(v);
    else k_blend_bwd<M, 256, kMM><<<grid, kBlock, 0, s>>>(v);
}
template <Mode M>
void launch_bwd_single(const ViewDesc &v, int nb, bool mm, hipStream_t s) {
    if (mm) launch_bwd_single<M, true>(v, nb, s);
    else launch_bwd_single<M, false>(v, nb, s);
}

// `all`: the plan's views are scanned in full (GSB_FULL_SCAN), in batches of at most kAllBatchFwd.
template <Mode M>
const void *fwd_batched_fn(int nb, bool all) {
    if (all && nb == 64) return reinterpret_cast<const void *>(&k_blend_fwd_batched<M, 64, true>);
    if (all) return reinterpret_cast<const void *>(&k_blend_fwd_batched<M, kAllBatchFwd, true>);
    if (nb == 64) return reinterpret_cast<const void *>(&k_blend_fwd_batched<M, 64>);
    if (nb == 128) return reinterpret_cast<const void *>(&k_blend_fwd_batched<M, 128>);
    return reinterpret_cast<const void *>(&k_blend_fwd_batched<M, 256>);
}
template <Mode M, bool kMM>
const void *bwd_batched_fn(int nb) {
    if (nb == 64) return reinterpret_cast<const void *>(&k_blend_bwd_batched<M, 64, kMM>);
    if (nb == 128) return reinterpret_cast<const void *>(&k_blend_bwd_batched<M, 128, kMM>);
    return reinterpret_cast<const void *>(&k_blend_bwd_batched<M, 256, kMM>);
}
template <Mode M>
const void *bwd_batched_fn(int nb, bool mm) {
    return mm ? bwd_batched_fn<M, true>(nb) : bwd_batched_fn<M, false>(nb);
}
const void *batched_fn(gsb_precision prec, bool fwd, int nb, bool mm, bool all) {
    switch (prec) {
        case GSB_FP32_PLAIN: return fwd ? fwd_batched_fn<Mode::Plain>(nb, all) : bwd_batched_fn<Mode::Plain>(nb, mm);
        case GSB_FP16_GEMM: return fwd ? fwd_batched_fn<Mode::F16>(nb, all) : bwd_batched_fn<Mode::F16>(nb, mm);
        default: return fwd ? fwd_batched_fn<Mode::BF16>(nb, all) : bwd_batched_fn<Mode::BF16>(nb, mm);
    }
}

}  // namespace

ViewDesc make_view(int32_t W, int32_t H, const uint32_t *ranges, const uint32_t *point_list,
                   const float *means2d, const float *conics, const float *opacity,
                   const float *colors, int64_t n, const float bg[3]) {
    ViewDesc v{};
    v.W = W; v.H = H; v.gx = int32_t(grid_x(W));
    v.n_tiles = grid_x(W) * grid_y(H);
    v.ranges = ranges; v.point_list = point_list; v.n = n;
    v.means2d = means2d; v.conics = conics; v.opacity = opacity; v.colors = colors;
    v.bg[0] = bg[0]; v.bg[1] = bg[1]; v.bg[2] = bg[2];
    return v;
}

gsb_status blend_forward(const ViewDesc &v, gsb_precision prec, int nb, hipStream_t s) {
    if (!valid_batch(nb)) return fail(GSB_ERR_INVALID, "batch %d not in {64, 128, 256}", nb);
    switch (prec) {
        case GSB_FP32_PLAIN: launch_fwd_single<Mode::Plain>(v, nb, s); break;
        case GSB_FP16_GEMM: launch_fwd_single<Mode::F16>(v, nb, s); break;
        case GSB_BF16_GEMM: launch_fwd_single<Mode::BF16>(v, nb, s); break;
        default: return fail(GSB_ERR_INVALID, "unknown precision %d", int(prec));
    }
    return check_launch("blend_forward");
}

gsb_status blend_backward(const ViewDesc &v, gsb_precision prec, int nb, bool mm, hipStream_t s) {
    if (!valid_batch(nb)) return fail(GSB_ERR_INVALID, "batch %d not in {64, 128, 256}", nb);
    if (prec != GSB_FP32_PLAIN && prec != GSB_FP16_GEMM && prec != GSB_BF16_GEMM)
        return fail(GSB_ERR_INVALID, "unknown precision %d", int(prec));
    const unsigned gz = unsigned((v.n + 255) / 256);
    if (v.n > 0) k_zero_grads<<<dim3(gz, 1), 256, 0, s>>>(nullptr, v);
    switch (prec) {
        case GSB_FP32_PLAIN: launch_bwd_single<Mode::Plain>(v, nb, mm, s); break;
        case GSB_FP16_GEMM: launch_bwd_single<Mode::F16>(v, nb, mm, s); break;
        default: launch_bwd_single<Mode::BF16>(v, nb, mm, s); break;
    }
    if (v.n > 0) k_bwd_finish<<<dim3(gz, 1), 256, 0, s>>>(nullptr, v);
    return check_launch("blend_backward");
}

gsb_status pack_gaussians(const float *means2d, const float *conics, const float *opacity,
                          const float *colors, int64_t n, float *records, hipStream_t s) {
    if (n > 0)
        k_pack<<<dim3(unsigned((n + 255) / 256)), 256, 0, s>>>(
            reinterpret_cast<const float2 *>(means2d), reinterpret_cast<const F3 *>(conics),
            opacity, reinterpret_cast<const F3 *>(colors), n, reinterpret_cast<float4 *>(records));
    return check_launch("pack_gaussians");
}

template <Mode M>
static void launch_fwd_rec(const ViewDesc &v, dim3 grid, hipStream_t s) {
    if (few_tiles<M>(v.n_tiles))
        (v.reach ? k_blend_fwd_rec<M, true, false> : k_blend_fwd_rec<M, true, true>)<<<grid, kBlock, 0, s>>>(v);
    else
        (v.reach ? k_blend_fwd_rec<M, false, false> : k_blend_fwd_rec<M, false, true>)<<<grid, kBlock, 0, s>>>(v);
}

gsb_status blend_forward_packed(const ViewDesc &v, gsb_precision prec, hipStream_t s) {
    const dim3 grid(unsigned(xcd_grid(v.n_tiles)));
    switch (prec) {
        case GSB_FP32_PLAIN: launch_fwd_rec<Mode::Plain>(v, grid, s); break;
        case GSB_FP16_GEMM: launch_fwd_rec<Mode::F16>(v, grid, s); break;
        case GSB_BF16_GEMM: launch_fwd_rec<Mode::BF16>(v, grid, s); break;
        default: return fail(GSB_ERR_INVALID, "unknown precision %d", int(prec));
    }
    return check_launch("blend_forward_packed");
}

gsb_status blend_backward_packed(const ViewDesc &v, gsb_precision prec, hipStream_t s) {
    if (prec != GSB_FP32_PLAIN && prec != GSB_FP16_GEMM && prec != GSB_BF16_GEMM)
        return fail(GSB_ERR_INVALID, "unknown precision %d", int(prec));
    const unsigned gz = unsigned((v.n + 255) / 256);
    const dim3 grid(unsigned(xcd_grid(v.n_tiles)));
    if (v.n > 0) k_zero_grads<<<dim3(gz, 1), 256, 0, s>>>(nullptr, v);
    switch (prec) {
        case GSB_FP32_PLAIN: k_blend_bwd_rec<Mode::Plain><<<grid, kBlock, 0, s>>>(v); break;
        case GSB_FP16_GEMM: k_blend_bwd_rec<Mode::F16><<<grid, kBlock, 0, s>>>(v); break;
        default: k_blend_bwd_rec<Mode::BF16><<<grid, kBlock, 0, s>>>(v); break;
    }
    if (v.n > 0) k_bwd_finish<<<dim3(gz, 1), 256, 0, s>>>(nullptr, v);
    return check_launch("blend_backward_packed");
}

// Deterministic-backward workspace: a row per list position, its number among its Gaussian's rows (then,
// for Gaussians with many, room to order them), the positions by Gaussian, per Gaussian its first and
// its number of rows, the scan's scratch, the Gaussians with many rows.
namespace {
struct DetLayout {
    size_t partial, seq, list, first, rows, scratch, large, end;
};
size_t al256(size_t b) { return (b + 255) & ~size_t(255); }
DetLayout det_layout(int64_t n, int64_t pairs) {
    const size_t P = size_t(pairs > 0 ? pairs : 1), N = size_t(n > 0 ? n : 1);
    DetLayout L;
    size_t o = 0;
    L.partial = o; o += al256(sizeof(float) * kDetStride * P);
    L.seq = o;     o += al256(sizeof(uint32_t) * P);
    L.list = o;    o += al256(sizeof(uint32_t) * P);
    L.first = o;   o += al256(sizeof(uint32_t) * N);
    L.rows = o;    o += al256(sizeof(uint32_t) * N);
    L.scratch = o; o += al256(offsets_scratch_bytes(int64_t(N)));
    L.large = o;   o += al256(sizeof(uint32_t) * (1 + P / kDetWaveRows));
    L.end = o;
    return L;
}
}  // namespace

size_t backward_det_workspace_bytes(int64_t n, int64_t pairs) { return det_layout(n, pairs).end; }

gsb_status blend_backward_det(const ViewDesc &v0, gsb_precision prec, int64_t pairs, void *ws,
                              hipStream_t s) {
    const DetLayout D = det_layout(v0.n, pairs);
    char *w = static_cast<char *>(ws);
    ViewDesc v = v0;
    v.det_partial = reinterpret_cast<float *>(w + D.partial);
    v.det_pairs = pairs;
    uint32_t *first = reinterpret_cast<uint32_t *>(w + D.first);
    uint32_t *rows = reinterpret_cast<uint32_t *>(w + D.rows);
    uint32_t *seq = reinterpret_cast<uint32_t *>(w + D.seq), *list = reinterpret_cast<uint32_t *>(w + D.list);
    uint32_t *large = reinterpret_cast<uint32_t *>(w + D.large);
    v.det_rows = rows;
    v.det_seq = seq;
    const int64_t m = std::max(pairs, v.n);
    if (m > 0) k_det_init<<<dim3(unsigned((m + 255) / 256)), 256, 0, s>>>(rows, v.n, seq, pairs, large);
    const dim3 grid(unsigned(xcd_grid(v.n_tiles)));
    switch (prec) {
        case GSB_FP32_PLAIN: k_blend_bwd_det<Mode::Plain><<<grid, kBlock, 0, s>>>(v); break;
        case GSB_FP16_GEMM: k_blend_bwd_det<Mode::F16><<<grid, kBlock, 0, s>>>(v); break;
        case GSB_BF16_GEMM: k_blend_bwd_det<Mode::BF16><<<grid, kBlock, 0, s>>>(v); break;
        default: return fail(GSB_ERR_INVALID, "unknown precision %d", int(prec));
    }
    if (pairs > 0 && v.n > 0) {
        counts_to_offsets(rows, first, v.n, w + D.scratch, s);
        k_det_place<<<dim3(unsigned((pairs + 1023) / 1024)), 256, 0, s>>>(v.point_list, seq, pairs, first,
                                                                         v.n, list, large);
        const int64_t per = 4 * kGatherPer, blocks = kDetBlocks + (v.n + per - 1) / per;
        k_det_gather<<<dim3(unsigned(blocks)), 256, 0, s>>>(
            DetOut{v.records, v.dL_dmeans2d, v.dL_dconics, v.dL_dopacity, v.dL_dcolors}, v.det_partial,
            first, rows, list, seq, large, pairs, v.n);
    } else if (v.n > 0) {
        k_zero_grads<<<dim3(unsigned((v.n + 255) / 256), 1), 256, 0, s>>>(nullptr, v);
    }
    return check_launch("blend_backward_deterministic");
}

// ------------------------------------------------------------------------------- plans
struct Plan {
    int device = 0;
    int n_views = 0;
    gsb_precision prec = GSB_FP16_GEMM;
    Tuning tune{};
    int64_t max_n = 0;
    bool all = false;               // every entry is staged (the views' reach is 0)
    ViewDesc *d_views = nullptr;    // device copy, plan order
    int64_t *d_prefix = nullptr;    // [8][n_views + 1]
    unsigned int *d_counters = nullptr;   // [16]: forward queues, backward queues
    int grid_fwd = 0, grid_bwd = 0;   // persistent grids
    int64_t grid_items = 0;            // one-shot grid: 8 x the longest queue
};

gsb_status plan_create(const ViewDesc *views, int n_views, gsb_precision prec, const Tuning &t,
                       Plan **out) {
    if (!valid_batch(t.batch_fwd) || !valid_batch(t.batch_bwd))
        return fail(GSB_ERR_INVALID, "batch sizes must be 64, 128 or 256");
    if (t.launch != kLaunchPersistent && t.launch != kLaunchGrid)
        return fail(GSB_ERR_INVALID, "launch mode %d unknown", t.launch);
    Plan *p = new Plan();
    p->n_views = n_views;
    p->prec = prec;
    p->tune = t;
    hipError_t e = hipGetDevice(&p->device);
    // heaviest-first: Gaussians per tile is proportional to the mean tile list length
    std::vector<int> order(n_views);
    for (int i = 0; i < n_views; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return double(views[a].n) / double(views[a].n_tiles) > double(views[b].n) / double(views[b].n_tiles);
    });
    std::vector<ViewDesc> ordered(n_views);
    for (int i = 0; i < n_views; ++i) {
        ordered[i] = views[order[i]];
        p->max_n = std::max(p->max_n, ordered[i].n);
    }
    p->all = n_views > 0 && ordered[0].reach == 0;           // (the precision's flag: the same for all)
    std::vector<int64_t> prefix(size_t(kXcds) * (n_views + 1), 0);
    for (int x = 0; x < kXcds; ++x) {
        int64_t run = 0;
        for (int k = 0; k < n_views; ++k) {
            prefix[size_t(x) * (n_views + 1) + k] = run;
            const int64_t T = ordered[k].n_tiles;
            run += T * (x + 1) / kXcds - T * x / kXcds;
        }
        prefix[size_t(x) * (n_views + 1) + n_views] = run;
        p->grid_items = std::max(p->grid_items, run * kXcds);
    }
    // one launch holds 2^32 - 1 threads; past that its grid would be cut short without an error
    if (p->grid_items > int64_t(0xffffffffu) / kBlock) p->tune.launch = kLaunchPersistent;
    if (e == hipSuccess) e = hipMalloc(&p->d_views, sizeof(ViewDesc) * size_t(n_views));
    if (e == hipSuccess) e = hipMalloc(&p->d_prefix, sizeof(int64_t) * prefix.size());
    if (e == hipSuccess) e = hipMalloc(&p->d_counters, sizeof(unsigned int) * 2 * kXcds);
    if (e == hipSuccess) e = hipMemcpy(p->d_views, ordered.data(), sizeof(ViewDesc) * size_t(n_views), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(p->d_prefix, prefix.data(), sizeof(int64_t) * prefix.size(), hipMemcpyHostToDevice);
    int cus = 0, occ_f = 0, occ_b = 0;
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_f, batched_fn(prec, true, t.batch_fwd, false, p->all), kBlock, 0);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_b, batched_fn(prec, false, t.batch_bwd, t.bwd_mm != 0, p->all), kBlock, 0);
    if (e != hipSuccess) {
        (void)plan_destroy(p);      // the creation error is the one reported
        return fail(GSB_ERR_HIP, "plan_create: %s", hipGetErrorString(e));
    }
    const int want = t.blocks_per_cu > 0 ? t.blocks_per_cu : 1 << 30;
    p->grid_fwd = cus * std::max(1, std::min(want, occ_f));
    p->grid_bwd = cus * std::max(1, std::min(want, occ_b));
    // a multiple of 8 keeps every XCD's queue served by the same number of blocks
    p->grid_fwd = (p->grid_fwd + kXcds - 1) / kXcds * kXcds;
    p->grid_bwd = (p->grid_bwd + kXcds - 1) / kXcds * kXcds;
    *out = p;
    return GSB_OK;
}

hipError_t plan_destroy(Plan *p) {
    if (!p) return hipSuccess;
    // every buffer is freed; the first failure is the one reported
    hipError_t e = hipSuccess;
    for (void *d : {static_cast<void *>(p->d_views), static_cast<void *>(p->d_prefix),
                    static_cast<void *>(p->d_counters)}) {
        if (!d) continue;
        const hipError_t f = hipFree(d);
        if (e == hipSuccess) e = f;
    }
    delete p;
    return e;
}

template <Mode M>
void launch_fwd_batched(const Queues &Q, int nb, const Plan &p, hipStream_t s) {
    if (p.tune.launch == kLaunchGrid) {
        const dim3 g(unsigned(p.grid_items));
        if (p.all)
            (nb == 64 ? k_blend_fwd_grid<M, 64, true> : k_blend_fwd_grid<M, kAllBatchFwd, true>)<<<g, kBlock, 0, s>>>(Q);
        else if (nb == 64) k_blend_fwd_grid<M, 64><<<g, kBlock, 0, s>>>(Q);
        else if (nb == 128) k_blend_fwd_grid<M, 128><<<g, kBlock, 0, s>>>(Q);
        else k_blend_fwd_grid<M, 256><<<g, kBlock, 0, s>>>(Q);
        return;
    }
    const int grid = p.grid_fwd;
    if (p.all)
        (nb == 64 ? k_blend_fwd_batched<M, 64, true>
                  : k_blend_fwd_batched<M, kAllBatchFwd, true>)<<<grid, kBlock, 0, s>>>(Q);
    else if (nb == 64) k_blend_fwd_batched<M, 64><<<grid, kBlock, 0, s>>>(Q);
    else if (nb == 128) k_blend_fwd_batched<M, 128><<<grid, kBlock, 0, s>>>(Q);
    else k_blend_fwd_batched<M, 256><<<grid, kBlock, 0, s>>>(Q);
}
template <Mode M, bool kMM>
void launch_bwd_batched(const Queues &Q, int nb, const Plan &p, hipStream_t s) {
    if (p.tune.launch == kLaunchGrid) {
        const dim3 g(unsigned(p.grid_items));
        if (nb == 64) k_blend_bwd_grid<M, 64, kMM><<<g, kBlock, 0, s>>>(Q);
        else if (nb == 128) k_blend_bwd_grid<M, 128, kMM><<<g, kBlock, 0, s>>>(Q);
        else k_blend_bwd_grid<M, 256, kMM><<<g, kBlock, 0, s>>>(Q);
        return;
    }
    const int grid = p.grid_bwd;
    if (nb == 64) k_blend_bwd_batched<M, 64, kMM><<<grid, kBlock, 0, s>>>(Q);
    else if (nb == 128) k_blend_bwd_batched<M, 128, kMM><<<grid, kBlock, 0, s>>>(Q);
    else k_blend_bwd_batched<M, 256, kMM><<<grid, kBlock, 0, s>>>(Q);
}
template <Mode M>
void launch_bwd_batched(const Queues &Q, int nb, const Plan &p, hipStream_t s) {
    if (p.tune.bwd_mm) launch_bwd_batched<M, true>(Q, nb, p, s);
    else launch_bwd_batched<M, false>(Q, nb, p, s);
}

gsb_status plan_forward(Plan *p, hipStream_t s) {
    if (p->n_views == 0) return GSB_OK;
    Queues Q{p->d_views, p->d_prefix, p->d_counters, p->n_views};
    if (p->tune.launch == kLaunchPersistent) k_reset_counters<<<1, 64, 0, s>>>(p->d_counters, kXcds);
    switch (p->prec) {
        case GSB_FP32_PLAIN: launch_fwd_batched<Mode::Plain>(Q, p->tune.batch_fwd, *p, s); break;
        case GSB_FP16_GEMM: launch_fwd_batched<Mode::F16>(Q, p->tune.batch_fwd, *p, s); break;
        default: launch_fwd_batched<Mode::BF16>(Q, p->tune.batch_fwd, *p, s); break;
    }
    return check_launch("blend_batched_forward");
}

gsb_status plan_backward(Plan *p, hipStream_t s) {
    if (p->n_views == 0) return GSB_OK;
    Queues Q{p->d_views, p->d_prefix, p->d_counters + kXcds, p->n_views};
    const dim3 gz(unsigned((p->max_n + 255) / 256 > 0 ? (p->max_n + 255) / 256 : 1), unsigned(p->n_views));
    k_zero_grads<<<gz, 256, 0, s>>>(p->d_views, ViewDesc{});
    if (p->tune.launch == kLaunchPersistent)
        k_reset_counters<<<1, 64, 0, s>>>(p->d_counters + kXcds, kXcds);
    switch (p->prec) {
        case GSB_FP32_PLAIN: launch_bwd_batched<Mode::Plain>(Q, p->tune.batch_bwd, *p, s); break;
        case GSB_FP16_GEMM: launch_bwd_batched<Mode::F16>(Q, p->tune.batch_bwd, *p, s); break;
        default: launch_bwd_batched<Mode::BF16>(Q, p->tune.batch_bwd, *p, s); break;
    }
    k_bwd_finish<<<gz, 256, 0, s>>>(p->d_views, ViewDesc{});
    return check_launch("blend_batched_backward");
}

}  // namespace gsb
