// raster_fwd.hip -- the forward rasterizer.
//
// Sec. III-A, Eq. (3)-(4): every pixel composites, front to back in
// (depth, Gaussian index) order, the splats whose tile rectangle contains its
// tile: alpha = min(0.99, o exp(power)); splats with power > 0 or
// alpha < 1/255 are skipped; compositing stops before a splat that would
// take the transmittance below 1e-4; colour = sum c alpha T + T_final bg.
//
// MI355X design: a wavefront per 8 x 8 quadrant of a 16 x 16 tile, one pixel
// per lane, and a workgroup of two wavefronts per half tile.  A wave stages 64
// list entries at a time in LDS (list ids read coalesced, splat records
// gathered one batch ahead), keeping only the entries that can reach 1/255 in
// its quadrant (each lane bounds its own entry, then a ballot compacts the
// batch), and its inner loop runs the kept entries a few at a time, each a
// broadcast LDS read that feeds the lane's pixel evaluation of two FMAs and one
// v_exp_f32.  The waves walk the list independently and each stops as soon as
// its pixels are saturated; they meet once, to exchange their results through
// LDS, so that each writes four rows of 16 pixels.
//
// Bound by VALU issue.  A square quadrant meets fewer splats than a 16 x 4
// strip (539 against 601 kept entries per tile, summed over its four parts, at
// the benchmark view; 507 against 552 of them with a hit): 98.5 -> 89.2 us at
// 1008 x 756 with 200k splats, 83 -> 76 us at 1200 x 680 with 500k, 36 -> 31 us
// at 320 x 240 with 50k, 666 -> 598 us over 8 views of 1008 x 756 to 320 x 240
// with 1M; 426 -> 428 us over 4 views of 1008 x 756, where the outputs' traffic
// weighs more.  Without the exchange a wave writes rows of 8 pixels, and those
// half lines cost more than the square saves once the outputs outgrow the L2
// (515 us over the 4 views, 728 us over the 8).
//
// The inner loop tests only what can be: no clamp and no sign of the power in a
// batch of plain splats, and the two selects of a pixel that stops only when
// one does (428 -> 410 us over the 4 views, 598 -> 549 us over the 8).  More
// entries per step (4: 439 us) or fewer (1: 426 us) lose more in registers or
// LDS round trips; so do fewer resident waves (6 per SIMD: 422 us).
#include <type_traits>

#include "block_ops.h"
#include "raster_common.h"

namespace gsp {

constexpr int kQuad = kTile / 2;   // edge of a quadrant
constexpr int kFwdThreads = 2 * kWave;   // the two quadrants of a half tile

struct FwdArgs {
    const uint32_t *order;
    const uint2 *ranges;
    const uint32_t *vals;
    const float4 *geom;
    const float4 *color;
    float *tfinal;
    uint32_t *ncontrib;
    uint32_t *tile_last;   // [total_tiles][kSplitFwd]: largest contributor count of the quadrant
    uint32_t *neval;    // STATS only: entries evaluated per pixel (up to the stop)
    uint32_t *nblend;   // STATS only: entries blended per pixel
    float4 *ckpt;       // per cut and tile pixel: (T, colour in front of the cut)
    float *cfinal;      // [3][total_pix]: final colour, for tiles with cuts
    // L1-fused forward: each view's img holds dL/dimage of the mean absolute
    // error against the target its dl points to (instead of the image), and
    // with l1part each wave leaves the FP64 sum of |image - target| over the
    // 16 x 4 strip it writes at [tile * kSplitFwd + strip]
    double *l1part;
    int total_pix;
    int total_tiles;
    bool l1;
};

// STATS = true is a measurement variant that also counts, per pixel, the
// evaluated and blended (pixel, splat) pairs of the algorithm -- every list
// entry up to the pixel's stop counts as evaluated, culled or not; the work
// counts define the kernel's algorithmic operation count.
template <bool STATS>
__global__ __launch_bounds__(kFwdThreads) __attribute__((amdgpu_waves_per_eu(4)))
void k_raster_fwd(FwdArgs a, ViewsK views) {
    __shared__ StagedA stA[2][kBatch];
    __shared__ StagedB stB[2][kBatch];
    __shared__ StagedF stF[2][kBatch];
    __shared__ float out[4][kFwdThreads];   // colour, transmittance of the half's pixels, row by row
    __shared__ int out_last[kFwdThreads];
    int rank, half;
    half_of_block(blockIdx.x, rank, half);
    if (rank >= a.total_tiles) return;
    const int wv = threadIdx.x / kWave, quad = 2 * half + wv;
    StagedA *const sA = stA[wv];
    StagedB *const sB = stB[wv];
    StagedF *const sF = stF[wv];
    const int tile = (int)a.order[rank];
    const ViewK &vw = views.v[view_of_tile(views, tile)];
    const int lt = tile - vw.tile_base;
    const int tx = lt % vw.gw, ty = lt / vw.gw;
    const int px0 = vw.roi_x + kTile * tx, py0 = vw.roi_y + kTile * ty;
    const int lane = threadIdx.x & (kWave - 1);
    const int qx = kQuad * (quad & 1), qy = kQuad * (quad >> 1);   // the quadrant's first pixel in the tile
    const int lx = qx + (lane & (kQuad - 1)), ly = qy + lane / kQuad;
    const int rx = kTile * tx + lx, ry = kTile * ty + ly;

    // A pixel composites while its row offset fy is finite; one that stopped
    // (or lies outside the region) gets kInactiveRow, so that no later splat
    // is a candidate there.
    float T = 1.f, cr = 0.f, cg = 0.f, cb = 0.f;
    int last = 0;
    uint32_t ne = 0, nb = 0;
    const float fxl = (float)lx;
    float fy = rx < vw.roi_w && ry < vw.roi_h ? (float)ly : kInactiveRow;

    const uint2 rg = a.ranges[tile];
    const int len = (int)(rg.y - rg.x);

    // records of the batch being staged, gathered one batch ahead
    float4 g0, g1, gc;
    auto gather = [&](int k) {
        g0 = make_float4(0.f, 0.f, 0.f, 0.f);
        g1 = make_float4(-1.f, 0.f, -1.f, -INFINITY);   // inert: alpha = 0
        gc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < len) {
            const uint32_t id = a.vals[rg.x + k];
            g0 = a.geom[2 * (size_t)id];
            g1 = a.geom[2 * (size_t)id + 1];
            gc = a.color[id];
        }
    };
    // Cuts of the list for the backward's chunks (at multiples of kChunk):
    // at each cut the transmittance and accumulated colour of the pixels
    // still compositing are recorded, and the pixels that blend past the
    // first cut also store their final colour; the backward reads them only
    // for pixels that blend past the cut that ends its chunk.
    const int ncut = chunks_of(len) - 1;
    int cuts_done = 0;
    bool alive = wave_any(fy != kInactiveRow);   // some pixel still composites
    gather(lane);
    for (int b0 = 0; b0 < len; b0 += kBatch) {
        if (!alive) break;
        if (cuts_done < ncut && b0 == (cuts_done + 1) * kChunk) {
            // The lane index is read here, not reused from the kernel's
            // start, so that no per-lane record address stays live through
            // the compositing loop (it would cost the kernel a resident wave
            // per SIMD).
            uint32_t ln;
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
            if (fy != kInactiveRow)   // still compositing (so inside the region)
                a.ckpt[(size_t)((rg.x + (uint32_t)b0) / kChunk) * (kTile * kTile) +
                       (uint32_t)((qy + (int)(ln / kQuad)) * kTile + qx) + (ln & (kQuad - 1))] =
                    make_float4(T, cr, cg, cb);
            cuts_done++;
        }
        // Stage the entries that can reach 1/255 somewhere in this quadrant,
        // in list order; the others cannot change any of its pixels.
        const float u = rel_coord(g0.x, g0.z, px0), v = rel_coord(g0.y, g0.w, py0);
        const int k = b0 + lane;
        const float ul = u - (float)qx, vl = v - (float)qy;
        const bool keep = k < len && SplatForm(g1.x, g1.y, g1.z, g1.w)
                                         .reaches(ul - (float)(kQuad - 1), ul, vl - (float)(kQuad - 1), vl);
        const unsigned long long kept = __ballot(keep);
        const int nk = __popcll(kept);
        const bool plain_batch = __ballot(keep && !plain_splat(g1.x, g1.y, g1.z, g1.w)) == 0ull;
        if (keep) {
            const int r = kept_rank(kept);
            sA[r] = StagedA{u, v, g1.x, g1.y};
            sB[r] = StagedB{g1.z, g1.w, gc.x, gc.y};
            sF[r] = StagedF{gc.z, (uint32_t)k + 1u};
        }
        // padding up to the unroll width: inert records
        if (lane >= nk && lane < ((nk + kUnroll - 1) & ~(kUnroll - 1))) {
            sA[lane] = StagedA{0.f, 0.f, -1.f, 0.f};
            sB[lane] = StagedB{-1.f, -INFINITY, 0.f, 0.f};
            sF[lane] = StagedF{0.f, 0u};
        }
        wave_sync();
        gather(b0 + kBatch + lane);
        // PLAIN: no staged entry of the batch can reach the 0.99 clamp or a
        // positive power (same alphas and hits, two operations fewer per
        // pixel); false once every pixel of the quadrant has stopped
        auto walk = [&](auto plain_c) __attribute__((always_inline)) {
            constexpr bool PLAIN = decltype(plain_c)::value;
            for (int j0 = 0; j0 < nk; j0 += kUnroll) {
                StagedA es[kUnroll];
                StagedB et[kUnroll];
                StagedF ef[kUnroll];
    #pragma unroll
                for (int u2 = 0; u2 < kUnroll; u2++) {
                    es[u2] = sA[j0 + u2];
                    et[u2] = sB[j0 + u2];
                    ef[u2] = sF[j0 + u2];
                }
    #pragma unroll
                for (int u2 = 0; u2 < kUnroll; u2++) {
                    const int jp1 = (int)ef[u2].jp1;   // list position + 1
                    const ColTerms ct = col_terms(es[u2], fxl);
                    // hit: still compositing (finite fy; see kInactiveRow) with
                    // power <= 0 and alpha >= 1/255, by which the backward decides
                    // too.  (No bound on p2 first: the staging cull already dropped
                    // the entries that reach 1/255 nowhere in the quadrant.)
                    const float p2 = splat_p2(ct, et[u2].C2, es[u2].v - fy);
                    const float apre = splat_alpha_pre(p2, et[u2].lo);
                    const float alpha = PLAIN ? apre : fminf(kAlphaMax, apre);
                    const bool hit = (PLAIN | (p2 <= 0.f)) & (alpha >= kAlphaMin);
                    if (!wave_any(hit)) continue;   // nothing to do for the quadrant
                    // A pixel without a hit takes alpha = 0, which leaves its T
                    // and colour exactly as they are.
                    float ahit = hit ? alpha : 0.f;
                    float testT = T - ahit * T;   // T (1 - alpha)
                    bool blend = hit;
                    // T >= 1e-4 until here, so only a hit can take it below: once
                    // in a pixel's walk, handled aside
                    const bool stop = !(testT >= kTMin);
                    if (wave_any(stop)) {
                        ahit = stop ? 0.f : ahit;
                        testT = stop ? T : testT;
                        blend = blend && !stop;
                        fy = stop ? kInactiveRow : fy;
                        if (STATS) ne = stop ? (uint32_t)jp1 : ne;
                        alive = wave_any(fy != kInactiveRow);
                    }
                    if (STATS) nb += blend ? 1u : 0u;
                    const float wgt = ahit * T;
                    cr = fmaf(et[u2].r, wgt, cr);
                    cg = fmaf(et[u2].g, wgt, cg);
                    cb = fmaf(ef[u2].b, wgt, cb);
                    last = blend ? jp1 : last;
                    T = testT;
                }
                if (!alive) return false;
            }
            return true;
        };
        const bool more = plain_batch ? walk(std::true_type{}) : walk(std::false_type{});
        if (!more) break;
        wave_sync();
    }

    if (STATS && rx < vw.roi_w && ry < vw.roi_h) {
        const size_t pix = (size_t)vw.pix_base + (size_t)ry * vw.roi_w + rx;
        // a pixel that never stopped evaluated the whole list
        a.neval[pix] = fy == kInactiveRow ? ne : (uint32_t)len;
        a.nblend[pix] = nb;
    }
    const int deepest = wave_max(last);
    if (lane == 0) a.tile_last[(size_t)tile * kSplitFwd + quad] = (uint32_t)deepest;
    // Every wave of the half gets here (each loop above ends for itself), and
    // each writes a 16 x 4 strip of it.
    {
        const int at = (lane / kQuad) * kTile + lx;
        out[0][at] = cr + T * vw.bg[0];
        out[1][at] = cg + T * vw.bg[1];
        out[2][at] = cb + T * vw.bg[2];
        out[3][at] = T;
        out_last[at] = last;
    }
    __syncthreads();
    const int ox = kTile * tx + (int)(threadIdx.x % kTile);
    const int oy = kTile * ty + kQuad * half + (int)(threadIdx.x / kTile);
    const int P = vw.roi_w * vw.roi_h;
    // L1-fused: sign(image - target) / (3 P), as gsp_loss_l1 writes it
    const float l1_inv = 1.0f / (float)(3 * (int64_t)P);
    double l1sum = 0.0;
    if (ox < vw.roi_w && oy < vw.roi_h) {
        const size_t pix = (size_t)oy * vw.roi_w + ox;
        float *img = vw.img;
        const float fr = out[0][threadIdx.x], fg = out[1][threadIdx.x], fb = out[2][threadIdx.x];
        const float Tf = out[3][threadIdx.x];
        const int lastf = out_last[threadIdx.x];
        if (a.l1) {
            const float *tg = vw.dl;
            const float c3[3] = {fr, fg, fb};
#pragma unroll
            for (int ch = 0; ch < 3; ch++) {
                const float d = c3[ch] - tg[(size_t)ch * P + pix];
                img[(size_t)ch * P + pix] = d > 0.f ? l1_inv : (d < 0.f ? -l1_inv : 0.f);
                l1sum += fabs((double)d);
            }
        } else {
            img[pix] = fr;
            img[(size_t)P + pix] = fg;
            img[2 * (size_t)P + pix] = fb;
        }
        if (lastf > kChunk) {   // the backward's chunks derive the colour behind a cut from it
            a.cfinal[vw.pix_base + pix] = fr;
            a.cfinal[(size_t)a.total_pix + vw.pix_base + pix] = fg;
            a.cfinal[2 * (size_t)a.total_pix + vw.pix_base + pix] = fb;
        }
        a.tfinal[vw.pix_base + pix] = Tf;
        a.ncontrib[vw.pix_base + pix] = (uint32_t)lastf;
        if (vw.alpha) vw.alpha[pix] = 1.f - Tf;
    }
    if (a.l1part) {
        l1sum = wave_sum(l1sum);
        if (lane == 0) a.l1part[(size_t)tile * kSplitFwd + quad] = l1sum;   // strip 2 half + wv
    }
}

// Loss of an L1-fused forward: per view, the waves' partial sums in tile and
// strip order, over the view's 3 x roi_h x roi_w values.
__global__ __launch_bounds__(256) void k_l1_fused_final(ViewsK views, const double *l1part,
                                                        float *loss) {
    __shared__ double red[256 / kWave];
    const ViewK &vw = views.v[blockIdx.x];
    const int64_t b0 = (int64_t)vw.tile_base * kSplitFwd, n = (int64_t)vw.gw * vw.gh * kSplitFwd;
    double s = 0.0;
    for (int64_t k = threadIdx.x; k < n; k += 256) s += l1part[b0 + k];
    s = block_sum<double, 256>(s, red);
    if (threadIdx.x == 0) loss[blockIdx.x] = (float)(s / (double)(3 * (int64_t)vw.roi_w * vw.roi_h));
}

hipError_t launch_raster_fwd(const ViewsK &views, const Layout &L, char *ws, const uint32_t *vals,
                             bool stats, hipStream_t s, bool l1, float *loss) {
    if (L.total_tiles == 0) return hipSuccess;
    FwdArgs a;
    a.l1 = l1;
    a.l1part = l1 && loss ? region<double>(ws, L.l1part) : nullptr;
    a.order = region<uint32_t>(ws, L.tile_order);
    a.ranges = region<uint2>(ws, L.ranges);
    a.vals = vals;
    a.geom = region<float4>(ws, L.geom);
    a.color = region<float4>(ws, L.color);
    a.tfinal = region<float>(ws, L.tfinal);
    a.ncontrib = region<uint32_t>(ws, L.ncontrib);
    a.tile_last = region<uint32_t>(ws, L.tile_last);
    a.neval = region<uint32_t>(ws, L.stats);
    a.nblend = a.neval + L.total_pix;
    a.ckpt = region<float4>(ws, L.ckpt);
    a.cfinal = region<float>(ws, L.cfinal);
    a.total_pix = (int)L.total_pix;
    a.total_tiles = L.total_tiles;
    const dim3 grid(raster_fwd_blocks(L.total_tiles));
    if (stats)
        hipLaunchKernelGGL(k_raster_fwd<true>, grid, dim3(kFwdThreads), 0, s, a, views);
    else
        hipLaunchKernelGGL(k_raster_fwd<false>, grid, dim3(kFwdThreads), 0, s, a, views);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.l1part) return e;
    hipLaunchKernelGGL(k_l1_fused_final, dim3(views.count), dim3(256), 0, s, views, a.l1part, loss);
    return hipGetLastError();
}

}  // namespace gsp
