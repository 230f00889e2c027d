// raster_bwd.hip -- backward of the compositing of Eq. (3)-(4).
//
// For the blended entries i of a pixel, with upstream G = dL/dC and T_i the
// transmittance in front of i:
//   dL/dc_i     = G alpha_i T_i
//   dL/dalpha_i = T_i G . (c_i - S_i),  S_i = colour behind i seen through i,
//   S_last = bg,  S_{i-1} = alpha_i c_i + (1 - alpha_i) S_i
// and through alpha = o exp(power) (no gradient when clamped at 0.99):
//   dL/dpower = dL/dalpha alpha,  dL/do = dL/dpower / o,
//   dpower/du = -(A dx + B dy), dpower/dv = -(C dy + B dx),
//   dpower/dA = -dx^2/2, dpower/dB = -dx dy, dpower/dC = -dy^2/2.
//
// MI355X design: nothing per pixel is stored by the forward beyond T_final,
// the contributor count and, for lists that are cut, the final colour and
// (T, accumulated colour) at every cut.  The work items are (tile, chunk)
// pairs, so that no workgroup walks more than a chunk of a list that is cut
// (the longest lists would otherwise run alone at the end of the launch);
// one wavefront per item walks the chunk back to front from the largest
// contributor count of its pixels inside it, recovering
// T_i = T_{i+1} / (1 - alpha_i) with the forward's exact evaluation, and
// skips (per lane-parallel bound, as in the forward) the entries that reach
// 1/255 nowhere in the tile.  Each lane sums its pixels in registers; the
// nine sums are reduced over the 64 lanes in two steps: v_permlane32_swap
// and v_permlane16_swap leave each as 16 partial sums in one row of lanes (16
// VALU operations for the nine), which wait in LDS; every kPend entries, 9 kPend
// lanes each add up the 16 partials of one (entry, component) in a fixed
// order and store it into the instance's own slot (its position among the
// instances splat by splat), flagging it written.  No atomics: the per-splat
// sum over its slots happens later in a fixed order, so gradients are
// bit-reproducible.
//
// Bound by VALU issue: the VALUs are busy 93 % of the time over 4 views of
// 1008 x 756; some 75 % over one, whose last items leave the chip half empty for
// the last quarter of the kernel (chunks of 64 entries shorten that, but cost 10 %
// more over several views, whose items all read their pixels' state).
#include <cstring>
#include <type_traits>

#include "block_ops.h"
#include "raster_common.h"

namespace gsp {

constexpr int kPixPerLane = 4;   // pixels per lane, one column

struct BwdArgs {
    const uint32_t *items;   // work items tile * kMaxChunks + chunk, longest first
    const uint32_t *counters;
    const float4 *ckpt;
    const float *cfinal;
    int total_pix;
    const uint2 *ranges;
    const uint32_t *vals;
    const float4 *geom;
    const float4 *color;
    const uint2 *rect;
    const uint32_t *offsets;
    const float *tfinal;
    const uint32_t *ncontrib;
    const uint4 *tile_last;   // per tile: largest contributor count of each quadrant
    float *slots;          // [cap][9]
    uint8_t *slot_flags;   // [cap]: 1 where this kernel wrote the slot
    // stored-list variant only
    const uint32_t *order;     // tiles, longest list first
    const uint32_t *loff;      // [total_pix + 1] first pair of each pixel
    const PairRec *pairs;
    const uint32_t *lhdr;      // list header (overflow flag)
    int total_tiles;
};

constexpr uint32_t kNoSlot = 0xffffffffu;

// Slot of the instance of splat `id` in tile (tx, ty): its position splat by splat.
__device__ __forceinline__ uint32_t slot_of(const BwdArgs &a, uint32_t id, int tx, int ty) {
    const uint2 r = a.rect[id];
    const int x0 = r.x & 0xffff, y0 = r.x >> 16, x1 = r.y & 0xffff;
    return a.offsets[id] + (uint32_t)((ty - y0) * (x1 - x0) + (tx - x0));
}

// Pixel with no stored pair left, and the list position of padding records
// (never a pixel's next pair; below every pixel's count as a signed int, and
// the padding's empty band mask skips it in either walk).
constexpr uint32_t kNoPos = 0xffffffffu;
constexpr uint32_t kPadPos = 0xfffffffeu;

// STORED = false: the recomputing backward over (tile, chunk) work items.
// STORED = true: one workgroup per whole tile; each pixel's blended entries,
// with their alpha and the transmittance in front of them, come from the
// pair records the forward stored (GSP_STORE_LISTS); the walk, the
// culling, the gradient formulas and the reduction are the same.
// OPA = false (no opacity gradient wanted, e.g. a pose-only solve): the
// wave reduces eight sums per entry instead of nine (the opacity sum, which
// only the opacity gradient needs, is left out) and the slot's opacity
// component is written as zero.
// MANY chooses between two shapes of the same walk, with the same results: for
// many tiles one entry per step and five pending entries, which fit 84
// registers and 7.5 KB of LDS, five waves per SIMD; for few, where waves run
// alone and latency counts, two entries per step and seven pending ones (111
// registers, 9.1 KB, four waves).  (The stored-list variant spills with either's
// registers, and takes the first at four waves.)
template <bool STORED, bool OPA, bool MANY>
__global__ __launch_bounds__(kRasterThreads) __attribute__((amdgpu_waves_per_eu(MANY && !STORED ? 5 : 4)))
void k_raster_bwd(BwdArgs a, ViewsK views) {
    constexpr int kUnroll = MANY ? 1 : 2;   // entries whose LDS records are read together
    // Entries whose row partials wait in LDS before a flush (at most 7: nine
    // lanes per entry in the flush).
    constexpr int kPend = MANY ? 5 : 7;
    static_assert(9 * kPend <= kWave, "one flush lane per (entry, component)");
    __shared__ StagedA sA[kBatch];
    __shared__ StagedB sB[kBatch];
    __shared__ StagedC sC[kBatch];
    __shared__ uint32_t sM[kBatch];   // bands the entry may reach (band_mask)
    // Row partials of the nine sums of up to kPend entries (wave_sum9_rows),
    // register-major, rows kRowStride floats apart so that the lanes of a
    // flush, each reading its own row, spread over the banks; and the slot
    // and 1/o of each pending entry.
    constexpr int kRowStride = 17;
    constexpr int kRegStride = 4 * kRowStride;
    constexpr int kEntryStride = 3 * kRegStride;
    __shared__ float sP[kPend * kEntryStride];
    __shared__ uint32_t sPs[kPend];
    __shared__ float sPi[kPend];
    const int rank = blockIdx.x;
    uint32_t item;
    if (STORED) {
        if (rank >= a.total_tiles || a.lhdr[kListOverflow]) return;
        item = a.order[rank] * kMaxChunks;   // chunk 0 of an uncut walk
    } else {
        if ((uint32_t)rank >= a.counters[kCntItems]) return;
        item = a.items[rank];
    }
    const int tile = (int)(item / kMaxChunks), chunk = (int)(item % kMaxChunks);
    const ViewK &vw = views.v[view_of_tile(views, tile)];
    const int lt = tile - vw.tile_base;
    const int tx = lt % vw.gw, ty = lt / vw.gw;
    const int px0 = vw.roi_x + kTile * tx, py0 = vw.roi_y + kTile * ty;
    const int lane = threadIdx.x;
    const int lx = lane & 15, ly = lane >> 4;
    const int rx = kTile * tx + lx;
    const int P = vw.roi_w * vw.roi_h;

    // In a flush, lane k < 9 kPend sums component pc of pending entry pe,
    // whose row partials start at poff within the entry's area; pscale is
    // the component's scale (see the base-2 conic of raster_common.h; the
    // opacity's 1/o comes with the entry).
    const int pe = lane / 9, pc = lane % 9;
    const int pc8 = pc < 5 ? pc : pc - 1;   // position among the eight sums (pc != 5)
    const int poff = OPA ? ((pc == 8 ? 2 : pc >> 2) * 4 + sum9_row(pc)) * kRowStride
                         : ((pc8 >> 2) * 4 + sum9_row(pc8)) * kRowStride;
    const float pscale = pc == 0 || pc == 1 ? kLn2 : pc == 2 || pc == 4 ? -0.5f : pc == 3 ? -1.f : 1.f;
    int npend = 0;
    auto flush = [&]() {
        __syncthreads();   // one wavefront: orders the stashing stores before these loads
        if (lane < 9 * npend) {
            const float *src = sP + pe * kEntryStride + poff;
            float t[8];
#pragma unroll
            for (int i = 0; i < 8; i++) t[i] = src[i] + src[8 + i];
#pragma unroll
            for (int i = 0; i < 4; i++) t[i] += t[4 + i];
            const float sum = (t[0] + t[2]) + (t[1] + t[3]);
            const uint32_t slot = sPs[pe];
            if (slot != kNoSlot) {
                const float f = pc == 5 ? sPi[pe] : pscale;
                a.slots[9 * (size_t)slot + pc] = OPA || pc != 5 ? sum * f : 0.f;
                if (pc == 0) a.slot_flags[slot] = 1;
            }
        }
        __syncthreads();   // before the next entries overwrite the area
        npend = 0;
    };

    // GS = G . S: the upstream gradient dotted with the colour behind the
    // current splat, which is all that dL/dalpha needs of S.
    // This chunk holds list positions [clo, chi).  A pixel that composited
    // past chi starts at chi from the state the forward recorded at that
    // cut; the others start from their final state at their contributor
    // count, as in an unsplit walk.
    const uint2 rg = a.ranges[tile];
    const int len = (int)(rg.y - rg.x);
    const int nch = STORED ? 1 : chunks_of(len);
    const int clo = chunk * kChunk, chi = chunk == nch - 1 ? len : clo + kChunk;
    const float4 *const ck =
        chunk < nch - 1 ? a.ckpt + (size_t)((rg.x + (uint32_t)chi) / kChunk) * (kTile * kTile)
                        : nullptr;
    int maxlast = 0;
    if (!STORED) {
        // The largest contributor count of the tile's pixels in this chunk; none
        // when every pixel stopped in front of it, as in half of the items of
        // the joint and pose steps' long lists (they leave here, before their
        // pixels' state is read: 804 -> 783 us over 4 views of 1008 x 756,
        // 1027 -> 972 us over 8 views of three sizes).
        const uint4 tl = a.tile_last[tile];
        maxlast = min((int)max(max(tl.x, tl.y), max(tl.z, tl.w)), chi);
        if (maxlast <= clo) return;
    }
    // Batches of 64 entries ending at hi, walked back to front; positions
    // below clo are absent.  Records are gathered one batch ahead, by ids read
    // two batches ahead (so that no wave waits for the one to issue the other).
    float4 g0, g1, gc;
    uint32_t gslot, id = 0;
    auto read_id = [&](int k) {
        if (k >= clo) id = a.vals[rg.x + k];
    };
    auto gather = [&](int k) {
        g0 = make_float4(0.f, 0.f, 0.f, 0.f);
        g1 = make_float4(-1.f, 0.f, -1.f, -INFINITY);
        gc = make_float4(0.f, 0.f, 0.f, 0.f);
        gslot = kNoSlot;
        if (k >= clo) {
            g0 = a.geom[2 * (size_t)id];
            g1 = a.geom[2 * (size_t)id + 1];
            gc = a.color[id];
            gslot = slot_of(a, id, tx, ty);
        }
    };
    if (!STORED) {
        read_id(maxlast - kBatch + lane);
        gather(maxlast - kBatch + lane);
        read_id(maxlast - 2 * kBatch + lane);
    }
    float T[kPixPerLane], G[kPixPerLane][3], GS[kPixPerLane], fy[kPixPerLane];
    int last[kPixPerLane];
    // stored lists: the pixel's next pair back to front (position, alpha, T)
    // and its index; pbase is the pixel's first pair
    uint32_t npos[kPixPerLane], pidx[kPixPerLane], pbase[kPixPerLane];
    float nal[kPixPerLane];
#pragma unroll
    for (int q = 0; q < kPixPerLane; q++) {
        const int ryl = ly + 4 * q;
        const int ry = kTile * ty + ryl;
        const bool in = rx < vw.roi_w && ry < vw.roi_h;
        const size_t pix = (size_t)ry * vw.roi_w + rx;
        fy[q] = (float)ryl;
        if (STORED) {
            npos[q] = kNoPos;
            nal[q] = 0.f;
            T[q] = 1.f;
            pbase[q] = in ? a.loff[vw.pix_base + pix] : 0u;
            pidx[q] = in ? a.loff[vw.pix_base + pix + 1] : 0u;   // one past the last pair
            last[q] = 0;
            if (pidx[q] > pbase[q]) {
                pidx[q]--;
                const PairRec r = a.pairs[pidx[q]];
                npos[q] = r.pos;
                nal[q] = r.alpha;
                T[q] = r.T;
                last[q] = (int)r.pos + 1;
            }
        } else {
            T[q] = in ? a.tfinal[vw.pix_base + pix] : 1.f;
            last[q] = in ? (int)a.ncontrib[vw.pix_base + pix] : 0;
        }
        const float *dl = vw.dl;
        G[q][0] = in ? dl[pix] : 0.f;
        G[q][1] = in ? dl[(size_t)P + pix] : 0.f;
        G[q][2] = in ? dl[2 * (size_t)P + pix] : 0.f;
        float S0 = vw.bg[0], S1 = vw.bg[1], S2 = vw.bg[2];
        if (!STORED && last[q] > chi) {   // only when this chunk ends at a cut
            // final colour = colour in front of the cut + T_cut * colour behind it
            const float4 c = ck[ryl * kTile + lx];
            const size_t pf = (size_t)vw.pix_base + pix;
            const float inv = 1.f / c.x;
            T[q] = c.x;
            S0 = (a.cfinal[pf] - c.y) * inv;
            S1 = (a.cfinal[(size_t)a.total_pix + pf] - c.z) * inv;
            S2 = (a.cfinal[2 * (size_t)a.total_pix + pf] - c.w) * inv;
            last[q] = chi;
        }
        GS[q] = G[q][0] * S0 + G[q][1] * S1 + G[q][2] * S2;
        if (STORED) maxlast = max(maxlast, last[q]);
    }
    if (STORED) {
        maxlast = wave_max(maxlast);
        if (maxlast > clo) {
            read_id(maxlast - kBatch + lane);
            gather(maxlast - kBatch + lane);
            read_id(maxlast - 2 * kBatch + lane);
        }
    }
    // largest contributor count of each band: an entry at or past it has no
    // candidate pixel in the band
    int blast[kPixPerLane];
#pragma unroll
    for (int q = 0; q < kPixPerLane; q++) blast[q] = __builtin_amdgcn_readfirstlane(wave_max(last[q]));
    const float fxl = (float)lx;

    for (int hi = maxlast; hi > clo; hi -= kBatch) {
        const int lo = hi - kBatch;
        // Stage, in list order, the entries that can reach 1/255 somewhere in
        // the tile; a dropped entry blends nowhere there, and its slot
        // stays unwritten (flag 0, read as zero).
        const float u = rel_coord(g0.x, g0.z, px0), v = rel_coord(g0.y, g0.w, py0);
        const uint32_t mask =
            gslot != kNoSlot ? band_mask(u, v, g1.x, g1.y, g1.z, g1.w) : 0u;
        const unsigned long long kept = __ballot(mask != 0u);
        const int nk = __popcll(kept);
        const bool nc_batch = __ballot(mask != 0u && !(g1.w <= kLoNoClamp)) == 0ull;
        const bool plain_batch = __ballot(mask != 0u && !plain_splat(g1.x, g1.y, g1.z, g1.w)) == 0ull;
        if (mask != 0u) {
            const int r = kept_rank(kept);
            sA[r] = StagedA{u, v, g1.x, g1.y};
            sB[r] = StagedB{g1.z, g1.w, gc.x, gc.y};
            sC[r] = StagedC{gc.z, __builtin_amdgcn_exp2f(-g1.w), gslot, (uint32_t)(lo + lane)};
            sM[r] = mask;
        }
        const int nkr = (nk + kUnroll - 1) & ~(kUnroll - 1);
        if (lane >= nk && lane < nkr) {   // padding up to the unroll width: reaches no band
            sA[lane] = StagedA{0.f, 0.f, -1.f, 0.f};
            sB[lane] = StagedB{-1.f, -INFINITY, 0.f, 0.f};
            sC[lane] = StagedC{0.f, 0.f, kNoSlot, kPadPos};
            sM[lane] = 0u;
        }
        __syncthreads();
        if (lo > clo) {
            gather(lo - kBatch + lane);
            read_id(lo - 2 * kBatch + lane);
        }
        // NC: no staged entry of the batch can reach the 0.99 clamp; PLAIN: nor a
        // positive power.  Their tests then drop out of the walk (fewer
        // operations).  The walk without the clamp keeps its own arithmetic
        // where the power is tested too: its sums round once less.
        auto walk = [&](auto nc_c, auto plain_c) __attribute__((always_inline)) {
            constexpr bool NC = decltype(nc_c)::value, PLAIN = decltype(plain_c)::value;
            for (int j0 = nkr - kUnroll; j0 >= 0; j0 -= kUnroll) {
                StagedA es[kUnroll];
                StagedB et[kUnroll];
                StagedC ew[kUnroll];
                uint32_t em[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; u++) {
                    es[u] = sA[j0 + u];
                    et[u] = sB[j0 + u];
                    ew[u] = sC[j0 + u];
                    em[u] = sM[j0 + u];
                }
                // All records of the group are wanted in registers here: the
                // compiler would otherwise sink the later entries' loads
                // below the band test, a second LDS round trip per entry.
                // (Not in the stored-list variant, where it would cost spills.)
#pragma unroll
                for (int u = 0; u < (STORED ? 0 : kUnroll); u++)
                    asm volatile("" ::"v"(es[u].u), "v"(es[u].v), "v"(es[u].A2), "v"(es[u].B2),
                                 "v"(et[u].C2), "v"(et[u].lo), "v"(et[u].r), "v"(et[u].g), "v"(ew[u].b),
                                 "v"(ew[u].inv_o), "v"(ew[u].slot));
#pragma unroll
                for (int u = kUnroll - 1; u >= 0; u--) {
                    // the bands this entry may reach that still have pixels
                    // compositing at its list position (wave-uniform)
                    const int pos = __builtin_amdgcn_readfirstlane((int)ew[u].pm);
                    uint32_t bands = __builtin_amdgcn_readfirstlane(em[u]);
#pragma unroll
                    for (int q = 0; q < kPixPerLane; q++)
                        if (pos >= blast[q]) bands &= ~(1u << q);
                    if (bands == 0u) continue;
                    const StagedA &s = es[u];
                    const StagedB &t = et[u];
                    const ColTerms ct = col_terms(s, fxl);
                    const float col3[3] = {t.r, t.g, ew[u].b};
                    // Per lane, dx is the same for all its pixels, so the conic
                    // and centre gradients need only the moments sum dp, sum dp dy,
                    // sum dp dy^2 of dL/dpower over them.
                    float m0 = 0.f, my = 0.f, myy = 0.f, gc[3] = {0.f, 0.f, 0.f};
                    bool blended = false;
                    // q-th pixels of all lanes form a 16 x 4 band of the tile: a
                    // band with no candidate pixel is skipped as a whole; inside a
                    // band the update is branch-free, pixels that do not blend
                    // adding exact zeros.
#pragma unroll
                    for (int q = 0; q < kPixPerLane; q++) {
                        if (!((bands >> q) & 1u)) continue;
                        const float dy = s.v - fy[q];
                        // candidates: pixels that blend this entry, decided as
                        // the forward does (power <= 0, alpha >= 1/255), before
                        // their contributor count
                        float apre = 0.f, a0 = 0.f;
                        bool cand;
                        if (STORED) {
                            cand = npos[q] == (uint32_t)pos;
                        } else {
                            const float p2 = splat_p2(ct, t.C2, dy);
                            apre = splat_alpha_pre(p2, t.lo);
                            a0 = NC ? apre : fminf(kAlphaMax, apre);
                            cand = (pos < last[q]) & (PLAIN | (p2 <= 0.f)) & (a0 >= kAlphaMin);
                        }
                        if (__builtin_amdgcn_ballot_w64(cand) == 0ull) continue;
                        blended = true;
                        float alpha, wgt;
                        bool valid, unclamped;
                        if (STORED) {
                            // alpha and T_i of this pair as the forward left them
                            valid = cand;
                            alpha = valid ? fabsf(nal[q]) : 0.f;
                            unclamped = nal[q] >= 0.f;
                            wgt = valid ? alpha * T[q] : 0.f;
                        } else {
                            // A pixel that does not blend takes alpha = 0, which
                            // leaves T (times rcp(1) = 1), G.S (plus 0 * diff)
                            // and the sums (plus 0) exactly as they are.
                            valid = cand;
                            alpha = valid ? a0 : 0.f;
                            unclamped = NC || apre <= kAlphaMax;
                            T[q] = T[q] * __builtin_amdgcn_rcpf(1.f - alpha);
                            wgt = alpha * T[q];
                        }
                        const float Gc = fmaf(G[q][2], col3[2], fmaf(G[q][1], col3[1], G[q][0] * col3[0]));
                        const float diff = Gc - GS[q];
#pragma unroll
                        for (int ch = 0; ch < 3; ch++) gc[ch] = fmaf(G[q][ch], wgt, gc[ch]);
                        GS[q] = STORED ? (valid ? fmaf(alpha, diff, GS[q]) : GS[q]) : fmaf(alpha, diff, GS[q]);
                        // dL/dpower; zero where alpha is clamped at 0.99
                        const float dp = unclamped ? wgt * diff : 0.f;
                        if (STORED && valid) {
                            // step to the pixel's previous pair (if any)
                            npos[q] = kNoPos;
                            if (pidx[q] > pbase[q]) {
                                pidx[q]--;
                                const PairRec r = a.pairs[pidx[q]];
                                npos[q] = r.pos;
                                nal[q] = r.alpha;
                                T[q] = r.T;
                            }
                        }
                        const float dpy = dp * dy;
                        m0 += dp;
                        my += dpy;
                        myy = fmaf(dpy, dy, myy);
                    }
                    if (!blended) continue;
                    {
                        // dpower/du = -(A dx + B dy), dpower/dv = -(C dy + B dx),
                        // dpower/d(A, B, C) = -(dx^2 / 2, dx dy, dy^2 / 2), in the
                        // base-2 conic and before the per-component scale below
                        float acc[9];
                        acc[0] = fmaf(s.B2, my, 2.f * s.A2 * ct.dx * m0);
                        acc[1] = fmaf(2.f * t.C2, my, ct.bdx * m0);
                        acc[2] = ct.dx * ct.dx * m0;
                        acc[3] = ct.dx * my;
                        acc[4] = myy;
                        acc[5] = OPA ? m0 : gc[0];
                        acc[6] = OPA ? gc[0] : gc[1];
                        acc[7] = OPA ? gc[1] : gc[2];
                        acc[8] = gc[2];
                        float *const dst = sP + npend * kEntryStride + (lane >> 4) * kRowStride + (lane & 15);
                        float ra, rb;
                        if (OPA) {
                            float rc;
                            wave_sum9_rows(acc, ra, rb, rc);
                            dst[2 * kRegStride] = rc;
                        } else {
                            wave_sum8_rows(acc, ra, rb);
                        }
                        dst[0] = ra;
                        dst[kRegStride] = rb;
                        if (lane == 0) {
                            sPs[npend] = ew[u].slot;
                            sPi[npend] = ew[u].inv_o;
                        }
                        if (++npend == kPend) flush();
                    }
                }
            }
        };
        if (!STORED && plain_batch) walk(std::true_type{}, std::true_type{});
        else if (!STORED && nc_batch) walk(std::true_type{}, std::false_type{});
        else walk(std::false_type{}, std::false_type{});
        __syncthreads();
    }
    if (npend > 0) flush();
}

// Launches of more tiles than this take the MANY shape.  Time of the kernel in it
// against the other: 0.95 to 0.98 for 4800 to 12096 tiles (one to eight views),
// 0.97 to 1.00 for 3750 to 3888, 0.99 to 1.00 for 3312, 1.00 to 1.03 for 3024 (a
// view of 1008 x 756) and 3225 (1200 x 680), and 1.04 to 1.09 for 300 and 64, where
// a few work items run alone for much of the launch.  Between 1200 and 3000 tiles
// it goes by the lists more than by the tiles (0.96 to 1.03: eight views of 320 x
// 240 0.97, one of 640 x 480 0.96 to 1.08), which the host does not know.
constexpr int kManyTiles = 3584;

hipError_t launch_raster_bwd(const ViewsK &views, const Layout &L, char *ws, const uint32_t *vals,
                             bool want_opacity, hipStream_t s) {
    if (L.total_tiles == 0) return hipSuccess;
    BwdArgs a;
    std::memset(&a, 0, sizeof a);
    a.items = region<uint32_t>(ws, L.items);
    a.counters = region<uint32_t>(ws, L.counters);
    a.ckpt = region<float4>(ws, L.ckpt);
    a.cfinal = region<float>(ws, L.cfinal);
    a.total_pix = (int)L.total_pix;
    a.ranges = region<uint2>(ws, L.ranges);
    a.vals = vals;
    a.geom = region<float4>(ws, L.geom);
    a.color = region<float4>(ws, L.color);
    a.rect = region<uint2>(ws, L.rect);
    a.offsets = region<uint32_t>(ws, L.offsets);
    a.tfinal = region<float>(ws, L.tfinal);
    a.ncontrib = region<uint32_t>(ws, L.ncontrib);
    a.tile_last = region<uint4>(ws, L.tile_last);
    a.slots = region<float>(ws, L.slots);
    a.slot_flags = region<uint8_t>(ws, L.slot_flags);
    // Slots that no entry writes keep the flag 0 that the forward
    // stored and count as zero.  The set of written slots depends only on the
    // forward's state, so repeated backwards of one forward agree on it.
    // one workgroup per possible work item; those past the
    // item count of this call exit at once
    const bool many = L.total_tiles > kManyTiles;
    auto *kernel = want_opacity ? (many ? k_raster_bwd<false, true, true> : k_raster_bwd<false, true, false>)
                                : (many ? k_raster_bwd<false, false, true> : k_raster_bwd<false, false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)L.max_items), dim3(kRasterThreads), 0, s, a, views);
    return hipGetLastError();
}

hipError_t launch_raster_bwd_stored(const ViewsK &views, const Layout &L, char *ws,
                                    const uint32_t *vals, const ListLayout &Q, const char *lists,
                                    hipStream_t s) {
    if (L.total_tiles == 0) return hipSuccess;
    BwdArgs a;
    std::memset(&a, 0, sizeof a);
    a.counters = region<uint32_t>(ws, L.counters);
    a.total_pix = (int)L.total_pix;
    a.ranges = region<uint2>(ws, L.ranges);
    a.vals = vals;
    a.geom = region<float4>(ws, L.geom);
    a.color = region<float4>(ws, L.color);
    a.rect = region<uint2>(ws, L.rect);
    a.offsets = region<uint32_t>(ws, L.offsets);
    a.slots = region<float>(ws, L.slots);
    a.slot_flags = region<uint8_t>(ws, L.slot_flags);
    a.order = region<uint32_t>(ws, L.tile_order);
    char *lw = const_cast<char *>(lists);
    a.loff = region<uint32_t>(lw, Q.offsets);
    a.pairs = region<PairRec>(lw, Q.pairs);
    a.lhdr = region<uint32_t>(lw, Q.hdr);
    a.total_tiles = L.total_tiles;
    // one workgroup per tile, in the forward's launch order
    hipLaunchKernelGGL((k_raster_bwd<true, true, true>), dim3(L.total_tiles),
                       dim3(kRasterThreads), 0, s, a, views);
    return hipGetLastError();
}

}  // namespace gsp
