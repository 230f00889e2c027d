// raster_common.h -- per-pixel splat evaluation shared by the forward and
// backward rasterizers, so that the backward's recomputation takes exactly
// the forward's decisions (same operations in the same order).
//
// Sec. III-A, Eq. (3): alpha = o exp(power), power = -1/2 d^T Sigma_hat^-1 d
// with d = pixel - mu_hat and Sigma_hat^-1 = [[A, B], [B, C]] (the paper
// prints Sigma_hat where its inverse is meant), so
// power = -1/2 (A dx^2 + C dy^2) - B dx dy.
//
// The preprocess stores the conic pre-scaled to base 2,
// (A2, B2, C2) = -log2(e) (A/2, B, C/2), and lo = log2(o), so that
// p2 = log2(e) power = A2 dx^2 + B2 dx dy + C2 dy^2 and alpha = 2^(p2 + lo):
// two FMAs and one v_exp_f32 per pixel once the dx terms, which the pixels
// of a lane share (they lie in one column), are formed.
#pragma once

#include <hip/hip_runtime.h>

#include "gsp_internal.h"

namespace gsp {

// The forward gives each 8 x 8 quadrant of a 16 x 16 tile to a wavefront, one
// pixel per lane; the backward the whole tile, lane l owning pixels
// (l % 16, l / 16 + 4 q) for q < 4, so that its q-th pixels form the 16 x 4
// band q of the tile.  The forward's quadrants keep the SIMDs busy (a 1008 x
// 756 view has only 3024 tiles), and each walks, culls and stops for its own
// pixels.
constexpr int kRasterThreads = 64;
constexpr int kBatch = 64;          // list entries staged in LDS at a time
static_assert(kChunk % kBatch == 0, "the backward's chunks start at batch boundaries");
#ifndef GSP_FWD_UNROLL
#define GSP_FWD_UNROLL 2
#endif
constexpr int kUnroll = GSP_FWD_UNROLL;   // entries per step of the inner loop

constexpr float kLn2 = 0.6931471805599453f;
// A splat can reach alpha >= 1/255 at a pixel only if p2 + log2(o) is at least
// log2(1/255).  Both rasterizers decide by alpha >= 1/255 and p2 <= 0; this is the
// bound that entries are culled by (SplatForm) and the stored lists' walk tests
// first, as p2 >= this - log2(o).  The 0.01 margin keeps it conservative with
// respect to v_exp_f32's and the subtraction's rounding, so skipping on it never
// changes a decision.
constexpr float kLog2AlphaMinLoose = -7.994353436858858f - 0.01f;
// log2 of an opacity that keeps every unclamped alpha of its splat below the
// 0.99 clamp: exp2(-0.0155) = 0.98931, so with power <= 0 the alpha stays
// below 0.99 by far more than the error of the exp2 instruction, and
// min(0.99, alpha) is alpha itself.
constexpr float kLoNoClamp = -0.0155f;

// Splat as staged in LDS: centre relative to the tile's first pixel, scaled
// conic, log2 opacity and colour; the forward adds its list position + 1, the
// backward its list position, the instance's slot and 1/o.  Every lane reads
// every staged byte, so the forward's record is kept to 40 bytes.
struct StagedA { float u, v, A2, B2; };
struct StagedB { float C2, lo, r, g; };
struct StagedF { float b; uint32_t jp1; };
struct StagedC { float b, inv_o; uint32_t slot, pm; };   // pm: list position

// Row that marks a pixel as done: every splat's p2 there is -inf (alpha 0), +inf, or
// not a number where the form has no extent in y (C2 = 0), and the tests on alpha and
// on the power's sign fail without a separate flag.  Batches walked without the
// latter have C2 < 0.
constexpr float kInactiveRow = INFINITY;

// Centre of a splat relative to pixel (px0, py0), from its (hi, lo) pair.
__device__ __forceinline__ float rel_coord(float hi, float lo, int origin) {
#pragma clang fp contract(off)
    return (hi - (float)origin) + lo;
}

// Per (lane, splat) terms shared by the pixels of a lane (one column).
struct ColTerms {
    float dx, adx2, bdx;
};

__device__ __forceinline__ ColTerms col_terms(const StagedA &s, float px) {
#pragma clang fp contract(off)
    ColTerms t;
    t.dx = s.u - px;
    t.adx2 = (s.A2 * t.dx) * t.dx;
    t.bdx = s.B2 * t.dx;
    return t;
}

// log2(e) * power at a pixel with offset dy.
__device__ __forceinline__ float splat_p2(const ColTerms &t, float C2, float dy) {
#pragma clang fp contract(off)
    return __fmaf_rn(dy, __fmaf_rn(C2, dy, t.bdx), t.adx2);
}

// Pre-clamp opacity o * exp(power).
__device__ __forceinline__ float splat_alpha_pre(float p2, float lo) {
#pragma clang fp contract(off)
    return __builtin_amdgcn_exp2f(p2 + lo);
}

// A splat's quadratic form over rectangles of offsets (dx, dy) from its centre.
// p2 is homogeneous of degree two, so from a point with p2 <= 0 it only grows
// towards the centre: over a rectangle it is largest at the centre if that
// lies inside, and otherwise on the one or two edges that face it, where
// A, C < 0 make it concave and largest at the edge's clamped stationary point
// (this holds too where rounding left a long thin form indefinite, since a
// pixel with p2 > 0 is never blended).
// reaches() is true when some pixel of the rectangle may reach alpha >= 1/255:
// where p2 >= kLog2AlphaMinLoose - lo may hold, without which alpha stays below;
// false is a proof that it fails at every pixel.  The margin
// covers the float32 rounding of the conic, of this bound and of the
// rasterizer's evaluation: 0.02 plus 1e-5 times the largest magnitude the three
// terms of p2 take in the rectangle, some forty times the error of either
// three-operation evaluation.  (Bounding every pixel row of a band by itself
// took 40 operations per 16 x 4 band where this takes 16.)
struct SplatForm {
    float A2, B2, C2, thr, kx, ky;   // dx = kx dy (dy = ky dx): stationary in dx (dy)
    bool any;                        // not concave along the edges: no bound
    __device__ __forceinline__ SplatForm(float A, float B, float C, float lo) : A2(A), B2(B), C2(C) {
        any = !(A < 0.f) || !(C < 0.f);
        thr = kLog2AlphaMinLoose - lo;
        kx = -0.5f * B * __builtin_amdgcn_rcpf(A);
        ky = -0.5f * B * __builtin_amdgcn_rcpf(C);
    }
    // over dx in [xa, xb], dy in [ya, yb]
    __device__ __forceinline__ bool reaches(float xa, float xb, float ya, float yb) const {
        const float x0 = fminf(fmaxf(0.f, xa), xb), y0 = fminf(fmaxf(0.f, ya), yb);
        const float ys = fminf(fmaxf(ky * x0, ya), yb), xs = fminf(fmaxf(kx * y0, xa), xb);
        const float fx = fmaf(fmaf(C2, ys, B2 * x0), ys, A2 * x0 * x0);   // on the edge dx = x0
        const float fy = fmaf(fmaf(A2, xs, B2 * y0), xs, C2 * y0 * y0);   // on the edge dy = y0
        const float xm = fmaxf(fabsf(xa), fabsf(xb)), ym = fmaxf(fabsf(ya), fabsf(yb));
        const float mag = fabsf(A2) * xm * xm + fabsf(B2) * xm * ym + fabsf(C2) * ym * ym;
        return any || fmaxf(fx, fy) + fmaf(1e-5f, mag, 0.02f) >= thr;
    }
};

// True for a splat whose opacity keeps o exp(power) below the 0.99 clamp
// wherever power <= 0, and whose form is definite enough that splat_p2 is never
// positive in float32: with B^2 <= 4 A C (1 - 1e-4), the sum in it stays
// negative under the relative errors (2^-24 each) of its three roundings, and
// the last rounding keeps the sign.  The errors are relative only above the
// smallest normal numbers, hence the floor under A C: it leaves out splats of
// some 1e5 pixels in both directions, whose products underflow at offsets below
// 1e-12 pixels at most.  The rasterizers walk a batch of such splats without the
// two tests.
__device__ __forceinline__ bool plain_splat(float A2, float B2, float C2, float lo) {
    const float ac = A2 * C2;
    return (lo <= kLoNoClamp) & (A2 < 0.f) & (ac >= 1e-20f) & (B2 * B2 <= 3.9996f * ac);
}

// Bit q of the result is set when some pixel of the 16 x 4 band q of the tile
// may be reached; u, v: the centre relative to the tile's first pixel.
__device__ __forceinline__ uint32_t band_mask(float u, float v, float A2, float B2, float C2, float lo) {
    const SplatForm f(A2, B2, C2, lo);
    uint32_t mask = 0u;
#pragma unroll
    for (int q = 0; q < 4; q++)
        mask |= f.reaches(u - (float)(kTile - 1), u, v - (float)(4 * q + 3), v - (float)(4 * q)) ? 1u << q : 0u;
    return mask;
}

// Position of a lane's entry among the entries of its wavefront that are
// kept, counting lanes below it.
__device__ __forceinline__ int kept_rank(unsigned long long kept) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
}

// Forward workgroup -> (rank of the tile in launch order, half).  The two
// halves of a tile go to workgroups 8 apart, which the dispatcher places
// on the same XCD (workgroups are dealt round-robin over the 8 XCDs), so the
// later one finds the tile's splat records in that XCD's L2.
__device__ __forceinline__ void half_of_block(int b, int &rank, int &half) {
    rank = (b >> 4) * 8 + (b & 7);
    half = (b >> 3) & 1;
}

// Workgroups of a forward launch over `tiles` tiles (whole groups of 8; the
// extra ones exit at once).
inline int raster_fwd_blocks(int tiles) { return ((tiles + 7) / 8) * 16; }

__device__ __forceinline__ int view_of_tile(const ViewsK &views, int tile) {
    int v = 0;
    while (v + 1 < views.count && tile >= views.v[v + 1].tile_base) v++;
    return v;
}

}  // namespace gsp
