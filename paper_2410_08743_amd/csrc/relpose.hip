// relpose.hip -- relative pose estimation between two frames (Sec. III-D):
// the scene of frame t from its depth map (pixels on a stride grid
// unprojected through the intrinsics into isotropic Gaussians with the
// pixel's colour and, as scale, the mean distance to their three nearest
// neighbours), and the confidence-masked L1 of Eq. (20)-(21) that the pose
// of frame t+1 is solved against.
//
// The nearest neighbours come from a search over the pixel grid, with the
// distances that a test of every point would give.  The points outside a
// window of pixels around the query's lie beyond one of the four planes
// through the camera centre and the window's edges, so a window whose
// third-smallest distance is under the distance to the nearest of those planes
// holds the three neighbours; where that does not settle a point, the bounding
// boxes of blocks of pixels say which blocks can hold one.
#include <type_traits>

#include "block_ops.h"
#include "gsp_internal.h"

namespace gsp {

constexpr float kY0 = 0.28209479177387814f;   // degree-0 SH basis value
constexpr float kInvalidLogit = -30.f;        // opacity of a pixel without depth
constexpr float kInvalidScale = 0.01f;        // scale of a point without neighbours

// Pixel blocks of both kernels: 32 x 8 grid pixels, one thread each.
constexpr int kGridW = 32, kGridH = 8, kGridThreads = kGridW * kGridH;

__host__ __device__ inline dim3 grid_blocks(int nx, int ny) {
    return dim3((nx + kGridW - 1) / kGridW, (ny + kGridH - 1) / kGridH);
}

// Also leaves the bounding box of each block's valid points (empty: +inf to
// -inf) in box[2 block], box[2 block + 1].
__global__ __launch_bounds__(kGridThreads) void k_unproject(UnprojK a) {
    __shared__ float red[6][kGridThreads / kWave];
    const int i = blockIdx.x * kGridW + threadIdx.x % kGridW, j = blockIdx.y * kGridH + threadIdx.x / kGridW;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (i < a.nx && j < a.ny) {
        const int k = j * a.nx + i;
        const int x = i * a.stride, y = j * a.stride;
        const size_t pix = (size_t)y * a.w + x;
        const float d = a.depth[pix];
        const bool ok = isfinite(d) && d > 0.f;
        const float z = ok ? d : 1.f;
        const float X = ((float)(x + a.roi_x) + 0.5f - a.cx) / a.fx * z;
        const float Y = ((float)(y + a.roi_y) + 0.5f - a.cy) / a.fy * z;
        a.means[3 * (size_t)k] = X;
        a.means[3 * (size_t)k + 1] = Y;
        a.means[3 * (size_t)k + 2] = z;
        a.quats[4 * (size_t)k] = 1.f;
        a.quats[4 * (size_t)k + 1] = 0.f;
        a.quats[4 * (size_t)k + 2] = 0.f;
        a.quats[4 * (size_t)k + 3] = 0.f;
        a.logits[k] = ok ? a.logit : kInvalidLogit;
        const size_t plane = (size_t)a.w * a.h;
        float *sh = a.sh + (size_t)k * 3 * a.S;
#pragma unroll
        for (int c = 0; c < 3; c++) sh[c] = (a.image[c * plane + pix] - 0.5f) / kY0;
        for (int e = 3; e < 3 * a.S; e++) sh[e] = 0.f;
        a.pts[k] = make_float4(X, Y, z, ok ? 1.f : 0.f);
        if (ok) {
            lo[0] = hi[0] = X;
            lo[1] = hi[1] = Y;
            lo[2] = hi[2] = z;
        }
    }
#pragma unroll
    for (int c = 0; c < 3; c++) {
        for (int off = kWave / 2; off > 0; off >>= 1) {
            lo[c] = fminf(lo[c], __shfl_xor(lo[c], off, kWave));
            hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], off, kWave));
        }
        if (threadIdx.x % kWave == 0) {
            red[c][threadIdx.x / kWave] = lo[c];
            red[3 + c][threadIdx.x / kWave] = hi[c];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const size_t blk = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
#pragma unroll
        for (int w = 1; w < kGridThreads / kWave; w++)
#pragma unroll
            for (int c = 0; c < 3; c++) {
                lo[c] = fminf(lo[c], red[c][w]);
                hi[c] = fmaxf(hi[c], red[3 + c][w]);
            }
        a.box[2 * blk] = make_float4(lo[0], lo[1], lo[2], 0.f);
        a.box[2 * blk + 1] = make_float4(hi[0], hi[1], hi[2], 0.f);
    }
}

__device__ __forceinline__ float distance2(float x, float y, float z, const float4 &q) {
    const float dx = x - q.x, dy = y - q.y, dz = z - q.z;
    return fmaf(dz, dz, fmaf(dy, dy, dx * dx));
}

// The three smallest squared distances seen, b0 <= b1 <= b2.
struct Near3 {
    float b0, b1, b2;
    __device__ __forceinline__ void insert(float d2) {
        const float n0 = fminf(b0, d2);
        const float n1 = fminf(b1, fmaxf(b0, d2));
        const float n2 = fminf(b2, fmaxf(b1, d2));
        b0 = n0;
        b1 = n1;
        b2 = n2;
    }
    __device__ __forceinline__ void test(const float4 &p, const float4 &q, bool other) {
        const float d2 = distance2(p.x, p.y, p.z, q);
        insert(p.w != 0.f && other ? d2 : INFINITY);
    }
};

// A number below the squared distance from the point q of grid pixel (i, j)
// to every point of a pixel more than r grid steps away in x or y: the
// squared distance to the nearest of the planes X = (a -+ d) Z, Y = (b -+ e) Z
// (a, b the pixel's ray, d, e the offset of the nearest ray outside the
// window; sides without pixels left do not count).  The 1e-3 and 1e-6 parts
// taken off the offset are hundreds of times the rounding of the rays and the
// points; a bound that this takes below zero says nothing (returns 0).
__device__ __forceinline__ float outside_bound(const UnprojK &a, const float4 &q, int i, int j, int r) {
    float lb = INFINITY;
    auto side = [&](bool exists, float ray, float step, float sign) {
        if (!exists) return;
        const float edge = ray + sign * step;
        const float d = step * 0.999f - 1e-6f * (1.f + fabsf(ray) + step);
        const float at = q.z * d * 0.9999f / sqrtf(fmaf(edge, edge, 1.f));
        lb = fminf(lb, at > 0.f ? at : 0.f);   // not a number: no bound
    };
    const float ra = ((float)(i * a.stride + a.roi_x) + 0.5f - a.cx) / a.fx;
    const float rb = ((float)(j * a.stride + a.roi_y) + 0.5f - a.cy) / a.fy;
    const float sx = (float)(r + 1) * (float)a.stride / a.fx, sy = (float)(r + 1) * (float)a.stride / a.fy;
    side(i - r > 0, ra, sx, -1.f);
    side(i + r < a.nx - 1, ra, sx, 1.f);
    side(j - r > 0, rb, sy, -1.f);
    side(j + r < a.ny - 1, rb, sy, 1.f);
    return lb * lb;
}

// log of the mean distance of each point to its three nearest valid
// neighbours (itself excluded), written to all three log scales.
//
// One thread per point tests the 7 x 7 pixels around it, staged in LDS with
// their halo (a step smaller leaves a fifth of the points of a noisy depth
// map to the second part).  Where the bound above does not settle a point --
// depth steps, holes, strong noise -- one of the block's waves searches for it
// (shared out, since they cluster: 37 us with each wave taking its own): a lane per
// block of pixels finds the nearest box, then those not further than the third
// neighbour so far (a box's distance is computed like a point's and every
// step rounds monotonically, so it never exceeds that of a point inside),
// and the wave tests their blocks, 64 pixels at a time.
// Bound by latency: 51k points (1200 x 680 at stride 4, 1 % depth noise, 0.2 %
// holes) took 2.03 ms when all pairs were tested from LDS, 25 us now.  A block
// has four times the wavefronts that its points take, for the second part: the
// depth of a render leaves it a third of the points, and 200 blocks of four
// wavefronts took 441 us with it where these take some 140 (28 us above).
// Where most of a block's points are left to the second part and most blocks can
// hold a neighbour, all pairs take less (all_pairs below): 1.06 ms in all for depths
// spread over forty octaves pixel by pixel, 3.7 block by block.  A frame without
// any depth takes 0.05 ms; without the test for empty boxes every one was near
// (3.8 ms).
constexpr int kKnnR = 3;
constexpr int kKnnThreads = 1024;   // one point for each of the first kGridThreads
constexpr int kKnnLW = kGridW + 2 * kKnnR, kKnnLH = kGridH + 2 * kKnnR;

// Neighbours of `count` of the block's points among all: each wavefront takes all
// of them, four to a lane, and its share of the other points, which it reads as
// scalars (those that do not count lie at infinity).  Six operations make a
// distance and three keep the smallest: the middle one of three is one.  (With a
// point to a lane the wavefronts wait for their scalars: twice the time.)
__device__ __forceinline__ void all_pairs(const UnprojK &a, const float4 (&tile)[kKnnLH][kKnnLW],
                                          const uint16_t *who, int count, Near3 *found) {
    constexpr int kEach = kGridThreads / kWave, kParts = kKnnThreads / kWave;
    __shared__ Near3 three[kKnnThreads];
    const int lane = threadIdx.x % kWave, part = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int n = a.nx * a.ny;
    float4 q[kEach];
    int self[kEach];
    Near3 mine[kEach];
#pragma unroll
    for (int g = 0; g < kEach; g++) {
        const int src = who[min(g * kWave + lane, count - 1)];
        self[g] = ((int)blockIdx.y * kGridH + src / kGridW) * a.nx + (int)blockIdx.x * kGridW + src % kGridW;
        q[g] = tile[src / kGridW + kKnnR][src % kGridW + kKnnR];
        mine[g] = Near3{INFINITY, INFINITY, INFINITY};
    }
    auto walk = [&](int c0, int c1, auto with_self) __attribute__((always_inline)) {
        const float4 *const pts = a.pts;
#pragma unroll 4
        for (int c = c0; c < c1; c++) {
            const float4 p = pts[c];
            const float px = p.w != 0.f ? p.x : INFINITY;
#pragma unroll
            for (int g = 0; g < kEach; g++) {
                float d2 = distance2(px, p.y, p.z, q[g]);
                if (decltype(with_self)::value) d2 = c == self[g] ? INFINITY : d2;
                const float b1 = __builtin_amdgcn_fmed3f(mine[g].b0, mine[g].b1, d2);
                mine[g].b2 = __builtin_amdgcn_fmed3f(mine[g].b1, mine[g].b2, d2);
                mine[g].b0 = fminf(mine[g].b0, d2);
                mine[g].b1 = b1;
            }
        }
    };
    // the points themselves lie in the block's rows
    const int s0 = (int)blockIdx.y * kGridH * a.nx, s1 = min(n, s0 + kGridH * a.nx);
    const int c0 = (int)((int64_t)part * n / kParts), c1 = (int)((int64_t)(part + 1) * n / kParts);
    walk(c0, min(c1, s0), std::false_type{});
    walk(max(c0, s0), min(c1, s1), std::true_type{});
    walk(max(c0, s1), c1, std::false_type{});
#pragma unroll
    for (int g = 0; g < kEach; g++) {
        three[threadIdx.x] = mine[g];
        __syncthreads();
        if (part == 0) {
            Near3 all = mine[g];
            for (int k = 1; k < kParts; k++) {
                const Near3 o = three[k * kWave + lane];
                all.insert(o.b0);
                all.insert(o.b1);
                all.insert(o.b2);
            }
            if (g * kWave + lane < count) found[who[g * kWave + lane]] = all;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kKnnThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_knn3(UnprojK a) {
    __shared__ float4 tile[kKnnLH][kKnnLW];
    __shared__ int s_count;                   // points left to the second part
    __shared__ uint16_t s_open[kGridThreads]; // and their threads
    __shared__ float s_third[kGridThreads];
    __shared__ Near3 s_found[kGridThreads];
    __shared__ int s_tested;                  // blocks tested for the wavefronts' first points
    const int i0 = blockIdx.x * kGridW, j0 = blockIdx.y * kGridH;
    if (threadIdx.x == 0) s_count = s_tested = 0;
    for (int e = threadIdx.x; e < kKnnLW * kKnnLH; e += kKnnThreads) {
        const int y = e / kKnnLW, x = e - y * kKnnLW;
        const int i = i0 + x - kKnnR, j = j0 + y - kKnnR;
        const bool in = i >= 0 && i < a.nx && j >= 0 && j < a.ny;
        tile[y][x] = in ? a.pts[(size_t)j * a.nx + i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    const int tx = threadIdx.x % kGridW, ty = threadIdx.x / kGridW;
    const int i = i0 + tx, j = j0 + ty;
    const bool valid = threadIdx.x < kGridThreads && i < a.nx && j < a.ny;
    Near3 best{INFINITY, INFINITY, INFINITY};
    bool open = false;
    if (valid) {
        const float4 q = tile[ty + kKnnR][tx + kKnnR];
#pragma unroll 1   // a row's points in flight; all 48 would take more registers than there are
        for (int dy = -kKnnR; dy <= kKnnR; dy++)
#pragma unroll
            for (int dx = -kKnnR; dx <= kKnnR; dx++)
                best.test(tile[ty + kKnnR + dy][tx + kKnnR + dx], q, dx != 0 || dy != 0);
        open = !(best.b2 < outside_bound(a, q, i, j, kKnnR));
    }
    if (open) {
        const int k = atomicAdd(&s_count, 1);
        s_open[k] = (uint16_t)threadIdx.x;
        s_third[threadIdx.x] = best.b2;
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int nblk = gridDim.x * gridDim.y;
    // Where most of the block's points are open, the wavefronts' first ones tell how
    // many blocks there are to test for a point; the others go through all pairs where that takes less: 36 cycles for each
    // of the n points (four times nine operations, a sixteenth of the points to a
    // wavefront), against some 175 for each open point and block tested for it.
    constexpr int kWaves = kKnnThreads / kWave;
    const int count = s_count, rest = count - kWaves, n = a.nx * a.ny;
    int k = threadIdx.x / kWave, stop = count > kGridThreads / 2 ? kWaves : count;
    for (;;) {
        for (; k < stop; k += kWaves) {
            const int src = s_open[k];
            const int si = i0 + src % kGridW, sj = j0 + src / kGridW;
            const float4 qs = tile[src / kGridW + kKnnR][src % kGridW + kKnnR];
            float limit = s_third[src];   // not below the third distance
            Near3 mine{INFINITY, INFINITY, INFINITY};
            auto box_of = [&](int b) {
                const float4 lo = a.box[2 * b], hi = a.box[2 * b + 1];
                const float dx = fmaxf(fmaxf(lo.x - qs.x, qs.x - hi.x), 0.f);
                const float dy = fmaxf(fmaxf(lo.y - qs.y, qs.y - hi.y), 0.f);
                const float dz = fmaxf(fmaxf(lo.z - qs.z, qs.z - hi.z), 0.f);
                return fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            };
            auto test_block = [&](int b) {   // b is the same in every lane
                const int bx = b % (int)gridDim.x, by = b / (int)gridDim.x;
                const int x = bx * kGridW + lane % kGridW, y0 = by * kGridH + lane / kGridW;
                float4 p[kGridThreads / kWave];
#pragma unroll
                for (int k = 0; k < kGridThreads / kWave; k++) {
                    const int y = y0 + k * (kWave / kGridW);
                    p[k] = x < a.nx && y < a.ny ? a.pts[(size_t)y * a.nx + x] : make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
                for (int k = 0; k < kGridThreads / kWave; k++)
                    mine.test(p[k], qs, x != si || y0 + k * (kWave / kGridW) != sj);
                limit = fminf(limit, wave_reduce(mine.b2, [](float x, float y) { return fminf(x, y); }));
            };
            // the nearest block first: its points bring the limit down for a
            // query far from the surface its pixel's neighbours lie on
            float dmin = INFINITY;
            int first = 0;
            for (int b = lane; b < nblk; b += kWave) {
                const float d = box_of(b);
                if (d < dmin) {
                    dmin = d;
                    first = b;
                }
            }
#pragma unroll
            for (int off = kWave / 2; off > 0; off >>= 1) {
                const float od = __shfl_xor(dmin, off, kWave);
                const int ob = __shfl_xor(first, off, kWave);
                if (od < dmin || (od == dmin && ob < first)) {
                    dmin = od;
                    first = ob;
                }
            }
            first = __builtin_amdgcn_readfirstlane(first);
            // (a box at infinite distance, empty or too far for its square, holds no
            // neighbour; where all are, there is none)
            if (wave_lane(dmin, 0) < INFINITY) test_block(first);
            int tested = 1;
            for (int b0 = 0; b0 < nblk; b0 += kWave) {
                const bool other = b0 + lane < nblk && b0 + lane != first;
                const float box = other ? box_of(b0 + lane) : INFINITY;
                unsigned long long near = __ballot(box <= limit && box < INFINITY);
                while (near != 0ull) {
                    const int bit = __ffsll(near) - 1;
                    near &= near - 1ull;
                    if (__shfl(box, bit, kWave) > limit) continue;   // ruled out since
                    test_block(b0 + bit);
                    tested++;
                }
            }
            if (stop < count && lane == 0) atomicAdd(&s_tested, tested);
#pragma unroll
            for (int off = kWave / 2; off > 0; off >>= 1) {
                const float o0 = __shfl_xor(mine.b0, off, kWave), o1 = __shfl_xor(mine.b1, off, kWave),
                            o2 = __shfl_xor(mine.b2, off, kWave);
                mine.insert(o0);
                mine.insert(o1);
                mine.insert(o2);
            }
            if (lane == 0) s_found[src] = mine;
        }
        if (stop == count) break;
        stop = count;
        __syncthreads();
        if (4ll * n < (int64_t)rest * s_tested) {
            all_pairs(a, tile, s_open + kWaves, rest, s_found);
            break;
        }
    }
    __syncthreads();
    if (!valid) return;
    if (open) best = s_found[threadIdx.x];
    float sum = 0.f;
    int cnt = 0;
    if (best.b0 < INFINITY) { sum += sqrtf(best.b0); cnt++; }
    if (best.b1 < INFINITY) { sum += sqrtf(best.b1); cnt++; }
    if (best.b2 < INFINITY) { sum += sqrtf(best.b2); cnt++; }
    const float ls = logf(cnt > 0 ? sum / (float)cnt : kInvalidScale);
    float *const out = a.log_scales + 3 * ((size_t)j * a.nx + i);
    out[0] = ls;
    out[1] = ls;
    out[2] = ls;
}

size_t unproject_scratch_bytes(int nx, int ny) {
    const dim3 g = grid_blocks(nx, ny);
    return sizeof(float4) * ((size_t)nx * ny + 2 * (size_t)g.x * g.y);
}

hipError_t launch_unproject(const UnprojK &a, hipStream_t s) {
    const int n = a.nx * a.ny;
    if (n <= 0) return hipSuccess;
    const dim3 grid = grid_blocks(a.nx, a.ny);
    hipLaunchKernelGGL(k_unproject, grid, dim3(kGridThreads), 0, s, a);
    hipLaunchKernelGGL(k_knn3, grid, dim3(kKnnThreads), 0, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Masked L1 (Eq. (21)): loss[v] = sum over pixels and channels of
// M |pred - target|, grad = M sign(pred - target), M = [alpha > 0.99] with
// alpha = 1 - T_final the render's accumulated opacity (Eq. (20)); the mask
// is decided in FP64 on the FP32 alpha.
// ---------------------------------------------------------------------------
constexpr int kMaskItems = 4096;

int64_t masked_blocks(int64_t count) { return (count + kMaskItems - 1) / kMaskItems; }

__global__ __launch_bounds__(256) void k_masked_l1(MaskViewsK a, double *partial) {
    __shared__ double red[256 / kWave];
    int v = 0;
    while (v + 1 < a.V && (int64_t)blockIdx.x >= a.blk_base[v + 1]) v++;
    const int64_t P = a.pix[v], count = 3 * P;
    const float *pred = a.pred[v], *target = a.target[v], *alpha = a.alpha[v];
    float *grad = a.grad[v];
    const int64_t base = ((int64_t)blockIdx.x - a.blk_base[v]) * kMaskItems;
    double s = 0.0;
    // every load of the thread before its first store, and the pixel by a
    // comparison (e < 3 P) instead of a 64-bit
    // remainder (14.8 -> 11.8 us at 1200 x 680)
    constexpr int kPer = kMaskItems / 256;
    float d[kPer], al[kPer];
#pragma unroll
    for (int r = 0; r < kPer; r++) {
        const int64_t e = base + (int64_t)r * 256 + threadIdx.x;
        const int64_t pix = e - (e >= 2 * P ? 2 * P : (e >= P ? P : 0));
        al[r] = e < count ? alpha[pix] : 0.f;
        d[r] = e < count ? pred[e] - target[e] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < kPer; r++) {
        const int64_t e = base + (int64_t)r * 256 + threadIdx.x;
        if (e < count) {
            const bool m = (double)al[r] > 0.99;
            grad[e] = m ? (d[r] > 0.f ? 1.f : (d[r] < 0.f ? -1.f : 0.f)) : 0.f;
            s += m ? fabs((double)d[r]) : 0.0;
        }
    }
    if (partial) {
        s = block_sum<double, 256>(s, red);
        if (threadIdx.x == 0) partial[blockIdx.x] = s;
    }
}

__global__ __launch_bounds__(256) void k_masked_l1_final(MaskViewsK a, const double *partial,
                                                         float *loss) {
    __shared__ double red[256 / kWave];
    const int v = blockIdx.x;
    double s = 0.0;
    for (int64_t b = a.blk_base[v] + threadIdx.x; b < a.blk_base[v + 1]; b += 256) s += partial[b];
    s = block_sum<double, 256>(s, red);
    if (threadIdx.x == 0) loss[v] = (float)s;
}

hipError_t launch_masked_l1(const MaskViewsK &a, float *loss, void *scratch, hipStream_t s) {
    const int64_t nblk = a.blk_base[a.V];
    if (nblk <= 0) return hipSuccess;
    double *partial = loss ? static_cast<double *>(scratch) : nullptr;
    hipLaunchKernelGGL(k_masked_l1, dim3((unsigned)nblk), dim3(256), 0, s, a, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !loss) return e;
    hipLaunchKernelGGL(k_masked_l1_final, dim3(a.V), dim3(256), 0, s, a, partial, loss);
    return hipGetLastError();
}

}  // namespace gsp
