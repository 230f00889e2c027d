// binning.hip -- the instances of every tile: one (depth, splat) entry per
// tile that a projected splat touches, grouped by tile, and what later stages
// need of the grouping (tile ranges, the tiles' launch order, the backward's
// work items, the splats' gradient slots).
//
// A counting sort by tile without a sort.  The splats of a view, in index
// order, are cut into chunks; one workgroup per chunk (and window of tiles,
// below) counts in LDS how many of its splats touch each tile (k_bin_count).
// A scan over the chunks of every tile (k_bin_scan) turns the counts into the
// place of each chunk's entries in the tile's list, and the same workgroups
// walk their splats again and write the entries there (k_bin_scatter), at
// positions that LDS atomics hand out.  Entries of one chunk and tile come in
// any order, those of different chunks in index order; the per-tile depth sort
// that follows orders by (depth, splat), so the result does not depend on it.
//
// MI355X design: nearly every CU takes one chunk of a single view, and an entry
// is written once.  Workgroups go round-robin over the 8 XCDs, and the chunks
// of one XCD are neighbours in index order: a tile's list is then written in 8
// contiguous pieces of one XCD each, whose lines leave that XCD's L2 whole.
// A radix sort by tile id (scan, emission, two passes of three kernels, ranges
// and launch order: eleven launches that wrote and read every entry three
// times) took 66 us at 1.5M instances in one 1008 x 756 view, 414 us at 15.4M
// in four and 657 us at 22M in eight views; the three kernels here take 6.1 +
// 5.0 + 15.2, 21 + 6 + 108 and 32 + 8 + 178 us.  The first is bound by latency
// and its row atomics, the last by the LDS atomic, the depth's gather and the
// scattered store that each entry takes.
#include <cstring>

#include "block_ops.h"
#include "gsp_internal.h"

namespace gsp {

// Tiles of a window: as many as a workgroup counts in LDS (16 KB).  A view of
// more tiles is cut into windows of whole tile rows (or, above kBinTiles tiles
// in a row, pieces of one), each a contiguous range of tile ids, and a
// workgroup takes the part of its splats that lies in its window.
constexpr int kBinTiles = 4096;
struct BinWindow {
    int view;
    int x0, x1, y0, y1;   // tile columns and rows
    int t0, nt;           // global tile id of the first, and number of tiles
};

__host__ __device__ inline int2 bin_window_shape(int gw, int gh) {
    if (gw > kBinTiles) return make_int2(kBinTiles, 1);
    const int most = kBinTiles / gw, nwy = (gh + most - 1) / most;
    return make_int2(gw, (gh + nwy - 1) / nwy);   // windows of equal height
}

int bin_windows_of(int gw, int gh) {
    const int2 s = bin_window_shape(gw, gh);
    return ((gw + s.x - 1) / s.x) * ((gh + s.y - 1) / s.y);
}

struct BinArgs {
    const uint2 *rect;             // [vn] x0 | y0 << 16, x1 | y1 << 16
    const uint32_t *tiles;         // [vn] tiles touched
    const uint32_t *depth;         // [vn] depth key
    uint32_t *mat;                 // [chunks][total_tiles] counts, then starts in the tile's list
    uint32_t *total;               // [total_tiles] list lengths
    unsigned long long *gsum;      // [groups] entries of each group of kWave tiles
    unsigned long long *csum;      // [V][chunks] entries of each chunk
    uint32_t *cstart;              // [V][chunks] entries of the chunks in front of each
    uint32_t *offsets;             // [vn + 1] first slot of each view-Gaussian, then M
    uint2 *wstart;                 // [windows + 1] first view-Gaussian of each work window and its first slot
    uint32_t *counters;
    uint2 *ranges;                 // [total_tiles]
    uint32_t *order, *items;       // launch order of the tiles, backward work items
    uint2 *pairs;                  // [cap] (depth key, view * n + i) of each instance
    uint8_t *slot_flags;           // [cap], cleared here for slots < M
    unsigned long long cap;
    int n, V, chunks, chunk_splats, total_tiles, groups;
    // chunks with more entries in a window than a workgroup stages: first piece,
    // window, chunk, -; and, per such chunk, the entries written so far per tile of
    // the window (both in the gradient slots, which are the backward's)
    uint4 *heavy;
    uint32_t *written;             // [max_heavy][kBinTiles]
    uint32_t max_heavy;
    int windows;                   // of all views
    int first[GSP_MAX_VIEWS];      // first window of each view
};

// Window w of all; the lanes look at a view each for the one that has it (32
// views one after the other, whose sizes each wait for a scalar load, took 10 us).
__device__ __forceinline__ BinWindow bin_window(const BinArgs &a, const ViewsK &views, int w) {
    BinWindow b;
    if (a.windows == a.V) {   // one each
        const ViewK &vw = views.v[w];
        b.view = w;
        b.x0 = b.y0 = 0;
        b.x1 = vw.gw;
        b.y1 = vw.gh;
        b.t0 = vw.tile_base;
    } else {
        const int lane = threadIdx.x % kWave;
        b.view = __popcll(__ballot(lane < a.V && a.first[lane < a.V ? lane : 0] <= w)) - 1;
        const ViewK &vw = views.v[b.view];
        const int2 s = bin_window_shape(vw.gw, vw.gh);
        const int nwx = (vw.gw + s.x - 1) / s.x, k = w - a.first[b.view];
        b.x0 = (k % nwx) * s.x;
        b.y0 = (k / nwx) * s.y;
        b.x1 = min(b.x0 + s.x, vw.gw);
        b.y1 = min(b.y0 + s.y, vw.gh);
        b.t0 = vw.tile_base + b.y0 * vw.gw + b.x0;
    }
    b.nt = (b.y1 - b.y0) * (b.x1 - b.x0);
    return b;
}

// Workgroup -> (window, chunk): chunks / 8 neighbouring chunks to an XCD.
// chunk may lie past the last one (the grid has whole eights).
__device__ __forceinline__ void bin_block(const BinArgs &a, int b, int &window, int &chunk) {
    const int per = (a.chunks + 7) / 8;
    window = b / (8 * per);
    const int c = b - window * 8 * per;
    chunk = (c & 7) * per + (c >> 3);
}

// Tiles of a splat in a window: columns [x0, x1) and rows [y0, y1) relative to
// the window's (none: x1 <= x0 or y1 <= y0).
struct BinRect {
    int x0, x1, y0, y1;
    __device__ __forceinline__ bool any() const { return x1 > x0 && y1 > y0; }
};

// A splat as loaded: tiles it touches (0: none) and their rect.
struct BinSplat {
    uint32_t full;
    uint2 rect;
};

__device__ __forceinline__ BinSplat bin_fetch(const BinArgs &a, const BinWindow &w, int i, int end) {
    BinSplat p{0u, make_uint2(0u, 0u)};
    if (i < end) {
        const size_t idx = (size_t)w.view * a.n + i;
        p.full = a.tiles[idx];
        p.rect = a.rect[idx];
    }
    return p;
}

__device__ __forceinline__ BinRect bin_clip(const BinWindow &w, const BinSplat &p) {
    BinRect r;
    r.x0 = max((int)(p.rect.x & 0xffff), w.x0) - w.x0;
    r.y0 = max((int)(p.rect.x >> 16), w.y0) - w.y0;
    r.x1 = p.full > 0 ? min((int)(p.rect.y & 0xffff), w.x1) - w.x0 : 0;
    r.y1 = min((int)(p.rect.y >> 16), w.y1) - w.y0;
    return r;
}

constexpr int kBinStage = 32256;   // entries of a chunk (in a window) that are staged in LDS
constexpr int kBinPiece = 16384;   // entries of a piece of a chunk that has more (+- a splat's)

constexpr int kBinCountThreads = 512;

// mat[chunk][tile] = splats of the chunk that touch the tile; csum[view][chunk]
// = all entries of the chunk.  A splat adds 1 at its first and takes 1 off
// behind its last column in each of its rows, and a scan along the rows makes
// counts of that: two LDS atomics per row of a splat instead of one per tile
// found by a search (79 -> 25 us at 15.4M instances
// of 4 x 1M splats, 10.1 -> 8.5 us at 1.5M; 21 and 6.1 since a workgroup finds its
// window without a walk).
__global__ __launch_bounds__(kBinCountThreads) void k_bin_count(BinArgs a, ViewsK views) {
    constexpr int NT = kBinCountThreads;
    __shared__ int diff[kBinTiles];
    __shared__ unsigned long long red[NT / kWave];
    __shared__ uint32_t row;
    int wi, chunk;
    bin_block(a, blockIdx.x, wi, chunk);
    if (chunk >= a.chunks) return;
    const BinWindow w = bin_window(a, views, wi);
    const int t = threadIdx.x, lane = t % kWave, cols = w.x1 - w.x0, rows = w.y1 - w.y0;
    const int begin = chunk * a.chunk_splats, end = min(a.n, begin + a.chunk_splats);
    for (int k = t; k < w.nt; k += NT) diff[k] = 0;
    __syncthreads();
    unsigned long long sum = 0, own = 0;   // entries, and those in the window
#pragma unroll 2
    for (int i = begin + t; i < end; i += NT) {
        const BinSplat p = bin_fetch(a, w, i, end);
        sum += p.full;
        const BinRect r = bin_clip(w, p);
        if (r.any()) {
            own += (uint32_t)(r.x1 - r.x0) * (uint32_t)(r.y1 - r.y0);
            for (int y = r.y0; y < r.y1; y++) {
                atomicAdd(&diff[y * cols + r.x0], 1);
                if (r.x1 < cols) atomicAdd(&diff[y * cols + r.x1], -1);
            }
        }
    }
    __syncthreads();
    uint32_t *const out = a.mat + (size_t)chunk * a.total_tiles + w.t0;
    for (int y = t / kWave; y < rows; y += NT / kWave) {
        int run = 0;
        for (int x0 = 0; x0 < cols; x0 += kWave) {
            const int x = x0 + lane;
            const int v = run + wave_inclusive_scan(x < cols ? diff[y * cols + x] : 0);
            if (x < cols) out[y * cols + x] = (uint32_t)v;
            run = wave_lane(v, kWave - 1);
        }
    }
    own = block_sum<unsigned long long, NT>(own, red);
    if (w.x0 == 0 && w.y0 == 0) {   // the view's first window
        sum = block_sum<unsigned long long, NT>(sum, red);
        if (t == 0) a.csum[(size_t)w.view * a.chunks + chunk] = sum;
    }
    if (own > (unsigned long long)kBinStage) {
        // (counts past what the capacity has room for overflow it: the chunks are
        // not written then)
        if (t == 0) {
            const unsigned long long pieces = min((own + kBinPiece - 1) / kBinPiece, 1ull << 18);
            const unsigned long long at =
                atomicAdd(reinterpret_cast<unsigned long long *>(a.counters + kCntPieces), 1ull << 32 | pieces);
            row = (uint32_t)(at >> 32);
            if (row < a.max_heavy) a.heavy[row] = make_uint4((uint32_t)at, (uint32_t)wi, (uint32_t)chunk, 0u);
        }
        __syncthreads();
        if (row < a.max_heavy)
            for (int k = t; k < w.nt; k += NT) a.written[(size_t)row * kBinTiles + k] = 0u;
    }
}

// Exclusive scan of every tile's counts over the chunks, in place; list
// lengths and their sums over groups of 64 tiles.  A workgroup takes one group:
// a lane per tile, and the chunks shared out over the 16 wavefronts, whose
// counts are all loaded at once (one round of memory latency).  One more
// workgroup scans the chunks' sums and writes the counters that follow from
// them.
constexpr int kBinScanWaves = 16, kBinScanPer = (kBinChunks + kBinScanWaves - 1) / kBinScanWaves;
constexpr int kBinScanThreads = kBinScanWaves * kWave;

__device__ __forceinline__ void bin_chunk_starts(const BinArgs &a) {
    __shared__ unsigned long long scratch[kBinScanWaves];
    unsigned long long all = 0;
    const int count = a.V * a.chunks;
    for (int k0 = 0; k0 < count; k0 += kBinScanThreads) {
        const int k = k0 + (int)threadIdx.x;
        unsigned long long total;
        const unsigned long long e =
            all + block_exclusive_scan<unsigned long long, kBinScanThreads>(k < count ? a.csum[k] : 0ull, scratch, &total);
        if (k < count) a.cstart[k] = (uint32_t)e;   // read only when all of them fit
        all += total;
    }
    if (threadIdx.x == 0) {
        const bool ovf = all > a.cap;
        a.counters[kCntMLo] = (uint32_t)(all & 0xffffffffull);
        a.counters[kCntMHi] = (uint32_t)(all >> 32);
        a.counters[kCntOverflow] = ovf ? 1u : 0u;
        a.counters[kCntMEff] = ovf ? 0u : (uint32_t)all;
        if (ovf) a.counters[kCntSticky] = 1u;
        if (a.n == 0) a.counters[kCntWin] = 0u;
    }
}

__global__ __launch_bounds__(kBinScanThreads) void k_bin_scan(BinArgs a) {
    __shared__ uint32_t part[kBinScanWaves][kWave];
    if ((int)blockIdx.x == a.groups) {
        bin_chunk_starts(a);
        return;
    }
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int tile = blockIdx.x * kWave + lane;
    const bool in = tile < a.total_tiles;
    uint32_t *const col = a.mat + tile;
    uint32_t c[kBinScanPer], s = 0;
#pragma unroll
    for (int j = 0; j < kBinScanPer; j++) {
        const int k = w * kBinScanPer + j;
        c[j] = in && k < a.chunks ? col[(size_t)k * a.total_tiles] : 0u;
    }
#pragma unroll
    for (int j = 0; j < kBinScanPer; j++) s += c[j];
    part[w][lane] = s;
    __syncthreads();
    uint32_t e = 0, total = 0;
#pragma unroll
    for (int v = 0; v < kBinScanWaves; v++) {
        const uint32_t p = part[v][lane];
        e += v < w ? p : 0u;
        total += p;
    }
#pragma unroll
    for (int j = 0; j < kBinScanPer; j++) {
        const int k = w * kBinScanPer + j;
        if (in && k < a.chunks) col[(size_t)k * a.total_tiles] = e;
        e += c[j];
    }
    if (w == 0) {
        if (in) a.total[tile] = total;
        const unsigned long long g = wave_sum((unsigned long long)total);
        if (lane == 0) a.gsum[blockIdx.x] = g;
    }
}

// Launch order of the tiles: longest lists first (in buckets of 4 lengths up
// to 1024, which spread the same-address LDS atomics of the counting sort four
// times thinner than buckets of 16, and of 64 lengths above), so that the
// longest tiles do not start last and leave a tail.  No bucket holds lengths
// on both sides of 1024 or of 2048: the lists longer than that are a prefix.
// The same workgroup lists the backward work items (tile, chunk), also longest
// first by chunk length.  The orders only decide which workgroup takes which
// tile or chunk; every result is the same in any order.
constexpr int kOrderBuckets = 512;
constexpr int kBinScatterThreads = 1024;
constexpr int kOrderRounds = 4;   // tiles per thread whose lengths are loaded together

__host__ __device__ constexpr int order_bucket(int len) {
    const int up = len <= 1024 ? (len + 3) >> 2 : 257 + ((len - 1025) >> 6);
    return kOrderBuckets - 1 - (up < kOrderBuckets - 1 ? up : kOrderBuckets - 1);
}

struct OrderShared {
    uint32_t cnt[2][kOrderBuckets], base[2][kOrderBuckets];
    unsigned long long gstart[kOrderRounds * kBinScatterThreads / kWave];   // first entry of each group
    unsigned long long carry;
};

// Tile ranges, launch order, work items and counters, by one workgroup while
// the others write the entries.  With ovf the lists count as empty.
__device__ __forceinline__ void bin_order(const BinArgs &a, OrderShared &s, bool ovf) {
    // Full chunks all fall into one bucket; a wave adds its tiles' full
    // chunks there with one atomic (same-address LDS atomics serialise).
    constexpr int kFull = order_bucket(kChunk);
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    for (int k = t; k < kOrderBuckets; k += kBinScatterThreads) s.cnt[0][k] = s.cnt[1][k] = 0;
    if (t == 0) s.carry = 0;
    __syncthreads();
    constexpr int kStep = kBinScatterThreads * kOrderRounds, kGroups = kStep / kWave;
    // lengths of this thread's tiles in the step starting at k0 (-1 past the last tile)
    auto load = [&](int k0, int (&len)[kOrderRounds]) {
#pragma unroll
        for (int r = 0; r < kOrderRounds; r++) {
            const int k = k0 + r * kBinScatterThreads + t;
            len[r] = k < a.total_tiles ? (ovf ? 0 : (int)a.total[k]) : -1;
        }
    };
    // The next step's lengths and group sums are loaded before a step's work.
    int len[kOrderRounds], ahead[kOrderRounds];
    auto load_group = [&](int k0) {
        const int g = k0 / kWave + lane;
        return w == 0 && g < a.groups && !ovf ? a.gsum[g] : 0ull;
    };
    static_assert(kGroups == kWave, "a lane per group of a step");
    load(0, len);
    unsigned long long gs = load_group(0);
    for (int k0 = 0; k0 < a.total_tiles; k0 += kStep) {
        load(k0 + kStep, ahead);
        const unsigned long long gs_ahead = load_group(k0 + kStep);
        // first entry of each group of the step
        if (w == 0) {
            const unsigned long long run = s.carry, inc = wave_inclusive_scan(gs);
            s.gstart[lane] = run + inc - gs;
            if (lane == kWave - 1) s.carry = run + inc;
        }
        __syncthreads();
        uint32_t full = 0;   // this thread's full chunks in the step
#pragma unroll
        for (int r = 0; r < kOrderRounds; r++) {
            const int k = k0 + r * kBinScatterThreads + t;
            if (k - lane >= a.total_tiles) break;   // whole wave past the end
            const uint32_t l = len[r] > 0 ? (uint32_t)len[r] : 0u;
            const uint32_t first = (uint32_t)s.gstart[r * (kBinScatterThreads / kWave) + w] + wave_inclusive_scan(l) - l;
            if (len[r] < 0) continue;
            a.ranges[k] = l > 0 ? make_uint2(first, first + l) : make_uint2(0u, 0u);
            const int nch = chunks_of(len[r]);
            atomicAdd(&s.cnt[0][order_bucket(len[r])], 1u);
            atomicAdd(&s.cnt[1][order_bucket(len[r] - (nch - 1) * kChunk)], 1u);
            full += (uint32_t)(nch - 1);
        }
        const uint32_t wfull = wave_sum(full);
        if (lane == 0 && wfull > 0) atomicAdd(&s.cnt[1][kFull], wfull);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kOrderRounds; r++) len[r] = ahead[r];
        gs = gs_ahead;
    }
    // exclusive scans of the two bucket histograms: one wave, eight buckets per lane
    constexpr int kPer = kOrderBuckets / kWave;
    if (t < kWave) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            uint32_t c[kPer], x = 0;
#pragma unroll
            for (int j = 0; j < kPer; j++) {
                c[j] = s.cnt[h][kPer * lane + j];
                x += c[j];
            }
            const uint32_t inc = wave_inclusive_scan(x);
            uint32_t e = inc - x;
#pragma unroll
            for (int j = 0; j < kPer; j++) {
                s.base[h][kPer * lane + j] = e;
                e += c[j];
            }
            if (h == 1 && lane == kWave - 1) a.counters[kCntItems] = inc;
        }
        // lists in front of the bucket that ends at 1024 (2048)
        if (lane == 0) {
            a.counters[kCntOver1024] = s.base[0][order_bucket(1024)];
            a.counters[kCntOver2048] = s.base[0][order_bucket(2048)];
        }
    }
    load(0, len);
    __syncthreads();
    for (int k0 = 0; k0 < a.total_tiles; k0 += kStep) {
        load(k0 + kStep, ahead);
        uint32_t full = 0;
#pragma unroll
        for (int r = 0; r < kOrderRounds; r++) full += len[r] >= 0 ? (uint32_t)(chunks_of(len[r]) - 1) : 0u;
        const uint32_t wfull = wave_sum(full);
        uint32_t wb = 0;
        if (lane == 0 && wfull > 0) wb = atomicAdd(&s.base[1][kFull], wfull);
        wb = wave_lane(wb, 0);   // the wave's first full-chunk item
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int r = 0; r < kOrderRounds; r++) {
            const int k = k0 + r * kBinScatterThreads + t;
            if (k - lane >= a.total_tiles) break;
            const int nch = len[r] >= 0 ? chunks_of(len[r]) : 1;
            if (len[r] >= 0) {
                a.order[atomicAdd(&s.base[0][order_bucket(len[r])], 1u)] = (uint32_t)k;
                a.items[atomicAdd(&s.base[1][order_bucket(len[r] - (nch - 1) * kChunk)], 1u)] =
                    (uint32_t)(k * kMaxChunks + nch - 1);
            }
            // full chunks j of the wave's tiles, compacted by ballot so that
            // each store covers consecutive items
            for (int j = 0; j < kMaxChunks - 1; j++) {
                const unsigned long long m = __ballot(j < nch - 1);
                if (m == 0ull) break;
                if (j < nch - 1) a.items[wb + (uint32_t)__popcll(m & below)] = (uint32_t)(k * kMaxChunks + j);
                wb += (uint32_t)__popcll(m);
            }
        }
#pragma unroll
        for (int r = 0; r < kOrderRounds; r++) len[r] = ahead[r];
    }
}

// A batch of one splat per thread, those with entries packed together: where
// each one's entries start among the batch's, its clipped rect and its place in
// the batch; and, per thread, the packed splat that its share of the entries
// starts in.  The window's tiles: next position of this chunk's entries, first
// in `entry` (staged) or in the list; then what to add to a staged position
// for that in the list.
constexpr int kBinLocalBits = 20;        // bits of a splat within its chunk, above them the tile
static_assert(kBinTiles <= 1 << (32 - kBinLocalBits), "a tile's bits");
struct ScatterShared {
    uint32_t cur[kBinTiles];
    uint32_t off[kBinScatterThreads + 1];
    uint2 rect[kBinScatterThreads];          // x0 | width << 16, y0 | place << 16
    uint16_t start[kBinScatterThreads];
    uint2 pack[2][kBinScatterThreads / kWave];
    uint32_t scratch[kBinScatterThreads / kWave];
    unsigned long long scratch2[kBinScatterThreads / kWave];
    uint32_t part[3][kBinScatterThreads / kWave];
    uint32_t piece;
    uint32_t entry[kBinStage];
};

// x / d for x and d below 2^16: the quotient's distance from the next whole
// number is at least 1 / (2 d), far above the rounding of x * (1 / d).
__device__ __forceinline__ uint32_t small_div(uint32_t x, uint32_t d) {
    return (uint32_t)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)d));
}

// A batch's entries, `per` consecutive ones per thread: a walk along the
// splats' tiles, four at a time (the four positions are asked for before the
// first is waited for).  put(position, splat in the batch, tile in the window).
template <typename F>
__device__ __forceinline__ void bin_walk(ScatterShared &s, uint32_t cols, uint32_t total, uint32_t per,
                                         F &&put) {
    uint32_t e = threadIdx.x * per;
    const uint32_t end = min(e + per, total);
    if (e >= end) return;
    uint32_t j = s.start[threadIdx.x];
    uint2 r = s.rect[j];
    uint32_t next = s.off[j + 1], width = r.x >> 16, x = e - s.off[j], row = small_div(x, width);
    x -= row * width;
    row = (row + (r.y & 0xffff)) * cols + (r.x & 0xffff);
    while (e < end) {
        constexpr int kAhead = 4;
        uint32_t who[kAhead], tile[kAhead], pos[kAhead];
        const int n = (int)min((uint32_t)kAhead, end - e);
#pragma unroll
        for (int q = 0; q < kAhead; q++) {
            if (q < n) {
                if (e == next) {   // the next splat's first tile
                    j++;
                    r = s.rect[j];
                    next = s.off[j + 1];
                    width = r.x >> 16;
                    x = 0;
                    row = (r.y & 0xffff) * cols + (r.x & 0xffff);
                }
                who[q] = r.y >> 16;
                tile[q] = row + x;
                pos[q] = atomicAdd(&s.cur[row + x], 1u);
                e++;
                if (++x == width) {
                    x = 0;
                    row += cols;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < kAhead; q++)
            if (q < n) put(pos[q], who[q], tile[q]);
    }
}

// A batch's splat with entries (mine of them, the first at e0, the j-th packed
// one), for the walk: its place among the batch's entries, its tiles, and the
// threads whose shares start in it.
__device__ __forceinline__ void bin_pack(ScatterShared &s, const BinRect &r, uint32_t mine, uint32_t e0, uint32_t j,
                                         uint32_t per) {
    if (mine == 0u) return;
    s.off[j] = e0;
    s.rect[j] = make_uint2((uint32_t)r.x0 | (uint32_t)(r.x1 - r.x0) << 16, (uint32_t)r.y0 | threadIdx.x << 16);
    for (uint32_t q = (e0 + per - 1) / per; q * per < e0 + mine; q++) s.start[q] = (uint16_t)j;
}

// The heavy chunks' pieces, shared out over the workgroups as they come free.
// Piece p of a chunk is the splats whose first entry lies in the p-th kBinPiece
// entries of the chunk in its window (a splat has no more than the window's
// tiles).  It is walked twice: to count its entries per tile and reserve their
// places in the chunk's part of the lists, and to write them there.  Every
// workgroup comes to its end when the pieces are taken; none waits for another.
__device__ __forceinline__ void bin_pieces(const BinArgs &a, const ViewsK &views, ScatterShared &s, uint32_t pieces,
                                           uint32_t heavy) {
    constexpr int NT = kBinScatterThreads, kPer = kBinTiles / NT;
    const int t = threadIdx.x;
    for (;;) {
        __syncthreads();
        if (t == 0) s.piece = atomicAdd(a.counters + kCntNextPiece, 1u);
        __syncthreads();
        const uint32_t p = s.piece;
        if (p >= pieces) return;
        uint32_t h = 0;   // the last chunk whose first piece is p or before it
        for (uint32_t past = heavy; past - h > 1;) {
            const uint32_t mid = (h + past) / 2;
            if (a.heavy[mid].x <= p) h = mid;
            else past = mid;
        }
        const uint4 rec = a.heavy[h];
        const BinWindow w = bin_window(a, views, (int)rec.y);
        const int chunk = (int)rec.z, begin = chunk * a.chunk_splats, end = min(a.n, begin + a.chunk_splats);
        const uint32_t x0 = (p - rec.x) * kBinPiece, cols = (uint32_t)(w.x1 - w.x0);
        const uint32_t idc = (uint32_t)((size_t)w.view * a.n + begin);
        // where the chunk's entries of each tile start: the lists in front of the
        // window, those in front of the tile, and the chunks in front
        uint32_t front = 0, first[kPer], sum = 0;
        const int g0 = w.t0 / kWave;
        for (int g = t; g < g0; g += NT) front += (uint32_t)a.gsum[g];
        if (g0 * kWave + t < w.t0) front += a.total[g0 * kWave + t];
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int k = kPer * t + j;
            first[j] = sum + (k < w.nt ? a.mat[(size_t)chunk * a.total_tiles + w.t0 + k] : 0u);
            sum += k < w.nt ? a.total[w.t0 + k] : 0u;
            if (k < w.nt) s.cur[k] = 0u;
        }
        uint32_t all;
        front = block_sum<uint32_t, NT>(front, s.scratch) + block_exclusive_scan<uint32_t, NT>(sum, s.scratch, &all);
#pragma unroll 1
        for (int pass = 0; pass < 2; pass++) {
            uint32_t run = 0;
            for (int i0 = begin; i0 < end && (run < x0 || run - x0 < kBinPiece); i0 += NT) {
                const BinRect r = bin_clip(w, bin_fetch(a, w, i0 + t, end));
                const uint32_t area = r.any() ? (uint32_t)(r.x1 - r.x0) * (uint32_t)(r.y1 - r.y0) : 0u;
                uint32_t batch;
                const uint32_t e = run + block_exclusive_scan<uint32_t, NT>(area, s.scratch, &batch);
                run += batch;
                if (run <= x0) continue;
                const uint32_t mine = e >= x0 && e - x0 < kBinPiece ? area : 0u;
                unsigned long long both;   // entries and splats of the piece
                const unsigned long long at = block_exclusive_scan<unsigned long long, NT>(
                    (unsigned long long)mine << 32 | (mine > 0 ? 1u : 0u), s.scratch2, &both);
                const uint32_t total = (uint32_t)(both >> 32), per = (total + NT - 1) / NT;
                if (t == 0) s.off[(uint32_t)both] = total;
                bin_pack(s, r, mine, (uint32_t)(at >> 32), (uint32_t)at, per);
                __syncthreads();
                const uint32_t id0 = idc + (uint32_t)(i0 - begin);
                bin_walk(s, cols, total, per, [&](uint32_t pos, uint32_t k, uint32_t) {
                    if (pass == 1) a.pairs[pos] = make_uint2(a.depth[id0 + k], id0 + k);
                });
                __syncthreads();
            }
            if (pass == 0) {
#pragma unroll
                for (int j = 0; j < kPer; j++) {
                    const int k = kPer * t + j;
                    const uint32_t c = k < w.nt ? s.cur[k] : 0u;
                    if (c > 0u) s.cur[k] = front + first[j] + atomicAdd(&a.written[(size_t)h * kBinTiles + k], c);
                }
                __syncthreads();
            }
        }
    }
}

// Writes the entries of a chunk in a window to the tiles' lists.  The view's first
// window also has what goes by splat: the first slot of each splat's instances (in
// index order, rows of the rect outer and columns inner: the backward's gradient
// slots), the work windows of the slot reduction, and the cleared slot flags.  Splat
// k's entry sits at position h = k + offsets[k] of the sequence (splat, its
// instances, next splat, ...), the next at h + 1 + count; work window b starts at
// the first splat whose entry is at or after b kWindow.
//
// Entries of the same tile are brought together in LDS first, so that a store
// covers runs of them: written one by one, each would be a partial line of its
// own wherever the lists being written exceed the L2 (190 -> 121 us at 15.4M
// instances in 12096 lists, 108 by now; 97 -> 62 us at 6.7M in 9600, now 47).  A chunk with too many
// entries (neighbouring splats that are large: a scene in an order of its own)
// leaves them to all workgroups, in pieces: 300 splats over a whole 1008 x 756 view
// in front of 200k small ones take 56 us, and took 554 where that chunk's workgroup
// wrote them alone.
__device__ __forceinline__ void bin_chunk(const BinArgs &a, const ViewsK &views, ScatterShared &s, int wi, int chunk,
                                          bool ovf) {
    constexpr int NT = kBinScatterThreads, NW = NT / kWave;
    const int t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    const BinWindow w = bin_window(a, views, wi);
    // Everything the block needs before its splats, in one round of memory
    // latency: the lists in front of the window; the window's lists and this
    // chunk's place in each; the first splats.
    const int begin = chunk * a.chunk_splats, end = min(a.n, begin + a.chunk_splats);
    const uint32_t before = a.cstart[w.view * a.chunks + chunk];
    constexpr int kPer = kBinTiles / NT;
    uint32_t front = 0, c[kPer], row[kPer], cnt[kPer];
    {
        const int g0 = w.t0 / kWave;
        for (int g = t; g < g0; g += NT) front += (uint32_t)a.gsum[g];
        if (g0 * kWave + t < w.t0) front += a.total[g0 * kWave + t];   // less than a group
        const uint32_t *const lists = a.total + w.t0;
        const uint32_t *const mrow = a.mat + (size_t)chunk * a.total_tiles + w.t0;
        const uint32_t *const mnext = chunk + 1 < a.chunks ? mrow + a.total_tiles : lists;
#pragma unroll
        for (int j = 0; j < kPer; j++) {
            const int k = kPer * t + j;
            c[j] = k < w.nt ? lists[k] : 0u;
            row[j] = k < w.nt ? mrow[k] : 0u;
            cnt[j] = k < w.nt ? mnext[k] : 0u;   // minus row: this chunk's entries
        }
    }
    BinSplat p = bin_fetch(a, w, begin + t, end);
    if (ovf) return;

    // A batch's splats: entries in the window and how many splats have any,
    // summed over the wavefronts in front by `pack`.
    BinRect r;
    uint32_t mine, inc, full;
    unsigned long long has;
    auto announce = [&](int parity) {
        full = p.full;
        r = bin_clip(w, p);
        mine = r.any() ? (uint32_t)(r.x1 - r.x0) * (uint32_t)(r.y1 - r.y0) : 0u;
        has = __ballot(mine > 0);
        inc = wave_inclusive_scan(mine);
        if (lane == kWave - 1) s.pack[parity][wv] = make_uint2(inc, (uint32_t)__popcll(has));
    };
    announce(0);
    // sum of front, and the scans of the lists and of this chunk's entries
    // over the window, in the same exchange
    uint32_t sum = 0, msum = 0;
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        cnt[j] -= row[j];
        sum += c[j];
        msum += cnt[j];
    }
    const uint32_t sinc = wave_inclusive_scan(sum), minc = wave_inclusive_scan(msum);
    front = wave_sum(front);
    if (lane == kWave - 1) {
        s.part[0][wv] = sinc;
        s.part[1][wv] = minc;
        s.part[2][wv] = front;
    }
    __syncthreads();
    uint32_t e = sinc - sum, le = minc - msum, entries = 0;
#pragma unroll
    for (int v = 0; v < NW; v++) {
        e += (v < wv ? s.part[0][v] : 0u) + s.part[2][v];
        le += v < wv ? s.part[1][v] : 0u;
        entries += s.part[1][v];
    }
    const bool whose = entries <= (uint32_t)kBinStage;   // this workgroup's to write
    const bool staged = whose && a.chunk_splats <= 1 << kBinLocalBits;
    // c becomes what takes a staged position to that in the list
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        const int k = kPer * t + j;
        if (k < w.nt) s.cur[k] = staged ? le : e + row[j];
        const uint32_t len = c[j];
        c[j] = e + row[j] - le;
        e += len;
        le += cnt[j];
    }

    const bool first = w.x0 == 0 && w.y0 == 0;   // the view's first window
    const bool whole = first && w.x1 == views.v[w.view].gw && w.y1 == views.v[w.view].gh;
    const uint32_t cols = (uint32_t)(w.x1 - w.x0);
    const uint32_t idc = (uint32_t)((size_t)w.view * a.n + begin);   // the chunk's first view-Gaussian
    uint32_t at = before;
    int parity = 0;
    for (int i0 = begin; i0 < (whose || first ? end : begin); i0 += NT, parity ^= 1) {
        const int i = i0 + t;
        uint32_t total = 0, nj = 0, e0 = inc - mine, j = (uint32_t)__popcll(has & ((1ull << lane) - 1ull));
#pragma unroll
        for (int v = 0; v < NW; v++) {
            const uint2 q = s.pack[parity][v];
            e0 += v < wv ? q.x : 0u;
            j += v < wv ? q.y : 0u;
            total += q.x;
            nj += q.y;
        }
        const uint32_t per = (total + NT - 1) / NT;
        if (t == 0) s.off[nj] = total;
        bin_pack(s, r, mine, e0, j, per);
        const uint32_t splat_full = full;
        __syncthreads();
        p = bin_fetch(a, w, i + NT, end);
        const uint32_t j0 = (uint32_t)(i0 - begin);
        if (staged)
            bin_walk(s, cols, total, per, [&](uint32_t pos, uint32_t k, uint32_t tile) {
                s.entry[pos] = tile << kBinLocalBits | (j0 + k);
            });
        else if (whose)
            bin_walk(s, cols, total, per, [&](uint32_t pos, uint32_t k, uint32_t) {
                a.pairs[pos] = make_uint2(a.depth[idc + j0 + k], idc + j0 + k);
            });
        if (first) {
            if (!whole) e0 = block_exclusive_scan<uint32_t, NT>(splat_full, s.scratch, &total);
            e0 += at;
            at += total;
            if (i < end) {
                const unsigned long long k = (unsigned long long)idc + (unsigned)(i - begin);
                const unsigned long long e1 = (unsigned long long)e0 + splat_full, h = k + e0, h1 = h + 1 + splat_full;
                a.offsets[k] = e0;
                if (k == 0) a.wstart[0] = make_uint2(0u, 0u);
                for (unsigned long long b = h / kWindow + 1; b * kWindow <= h1; b++)
                    a.wstart[b] = make_uint2((uint32_t)k + 1, (uint32_t)e1);
                const unsigned long long vn = (unsigned long long)a.V * a.n;
                if (k == vn - 1) {
                    const unsigned long long nwin = (h1 + kWindow - 1) / kWindow;
                    if (nwin * kWindow > h1) a.wstart[nwin] = make_uint2((uint32_t)vn, (uint32_t)e1);
                    a.offsets[vn] = (uint32_t)e1;
                    a.counters[kCntWin] = (uint32_t)nwin;
                }
            }
        }
        announce(parity ^ 1);
        __syncthreads();
    }
    if (staged) {
#pragma unroll
        for (int j = 0; j < kPer; j++)
            if (kPer * t + j < w.nt) s.cur[kPer * t + j] = c[j];
        __syncthreads();
#pragma unroll 4
        for (uint32_t k = t; k < entries; k += NT) {
            const uint32_t x = s.entry[k], id = idc + (x & ((1u << kBinLocalBits) - 1u));
            a.pairs[s.cur[x >> kBinLocalBits] + k] = make_uint2(a.depth[id], id);
        }
    }
    if (first) {   // the flags of the chunk's slots
        const unsigned long long f0 = before, f1 = at;
        const unsigned long long v0 = min((f0 + 15) & ~15ull, f1), v1 = max(f1 & ~15ull, v0);
        for (unsigned long long k = f0 + t; k < v0; k += NT) a.slot_flags[k] = 0;
        for (unsigned long long k = v0 + 16ull * t; k < v1; k += 16ull * NT)
            *reinterpret_cast<uint4 *>(a.slot_flags + k) = make_uint4(0, 0, 0, 0);
        for (unsigned long long k = v1 + t; k < f1; k += NT) a.slot_flags[k] = 0;
    }
}

// Workgroup 0 orders the tiles; the others write a chunk's entries in a window
// each, and then share out the pieces of the heavy chunks.
__global__ __launch_bounds__(kBinScatterThreads) void k_bin_scatter(BinArgs a, ViewsK views) {
    __shared__ union {
        OrderShared o;
        ScatterShared s;
    } sh;
    const bool ovf = a.counters[kCntOverflow] != 0u;
    if (blockIdx.x == 0) {
        bin_order(a, sh.o, ovf);
        return;
    }
    int wi, chunk;
    bin_block(a, blockIdx.x - 1, wi, chunk);
    const uint32_t pieces = a.counters[kCntPieces], heavy = a.counters[kCntHeavy];
    if (chunk < a.chunks) bin_chunk(a, views, sh.s, wi, chunk, ovf);
    if (!ovf && pieces > 0u) bin_pieces(a, views, sh.s, pieces, heavy);
}

static BinArgs bin_args(const ViewsK &views, const Layout &L, char *ws) {
    BinArgs a;
    std::memset(&a, 0, sizeof a);
    a.rect = region<uint2>(ws, L.rect);
    a.tiles = region<uint32_t>(ws, L.tiles);
    a.depth = region<uint32_t>(ws, L.depth);
    a.mat = region<uint32_t>(ws, L.binmat);
    a.total = region<uint32_t>(ws, L.tiletotal);
    a.gsum = region<unsigned long long>(ws, L.groupsum);
    a.csum = region<unsigned long long>(ws, L.chunksum);
    a.cstart = region<uint32_t>(ws, L.chunkstart);
    a.offsets = region<uint32_t>(ws, L.offsets);
    a.wstart = region<uint2>(ws, L.wstart);
    a.counters = region<uint32_t>(ws, L.counters);
    a.ranges = region<uint2>(ws, L.ranges);
    a.order = region<uint32_t>(ws, L.tile_order);
    a.items = region<uint32_t>(ws, L.items);
    a.pairs = region<uint2>(ws, L.pairs);
    a.slot_flags = region<uint8_t>(ws, L.slot_flags);
    a.cap = (unsigned long long)L.cap;
    // a heavy chunk has more than kBinStage instances of the capacity's, which
    // bring 36 bytes of slots each: room for its counts and its record
    static_assert(36ll * kBinStage >= 4 * kBinTiles + 16, "a heavy chunk's share of the slots");
    a.max_heavy = (uint32_t)(L.cap / (kBinStage + 1));
    a.written = region<uint32_t>(ws, L.slots);
    a.heavy = reinterpret_cast<uint4 *>(a.written + (size_t)a.max_heavy * kBinTiles);
    a.n = (int)L.n;
    a.V = L.V;
    a.chunks = L.bin_chunks;
    a.chunk_splats = L.bin_chunk_splats;
    a.total_tiles = L.total_tiles;
    a.groups = (L.total_tiles + kWave - 1) / kWave;
    for (int v = 0; v < views.count; v++) {
        a.first[v] = a.windows;
        a.windows += bin_windows_of(views.v[v].gw, views.v[v].gh);
    }
    return a;
}

static unsigned bin_blocks(const BinArgs &a) { return (unsigned)a.windows * 8u * (unsigned)((a.chunks + 7) / 8); }

hipError_t launch_bin_count(const ViewsK &views, const Layout &L, char *ws, hipStream_t s) {
    const BinArgs a = bin_args(views, L, ws);
    if (bin_blocks(a) == 0) return hipSuccess;
    hipLaunchKernelGGL(k_bin_count, dim3(bin_blocks(a)), dim3(kBinCountThreads), 0, s, a, views);
    return hipGetLastError();
}

hipError_t launch_bin_scan(const ViewsK &views, const Layout &L, char *ws, hipStream_t s) {
    const BinArgs a = bin_args(views, L, ws);
    hipLaunchKernelGGL(k_bin_scan, dim3(a.groups + 1), dim3(kBinScanThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_bin_scatter(const ViewsK &views, const Layout &L, char *ws, hipStream_t s) {
    const BinArgs a = bin_args(views, L, ws);
    hipLaunchKernelGGL(k_bin_scatter, dim3(bin_blocks(a) + 1), dim3(kBinScatterThreads), 0, s, a, views);
    return hipGetLastError();
}

}  // namespace gsp
