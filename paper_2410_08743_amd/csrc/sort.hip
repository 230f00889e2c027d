// sort.hip -- the (tile, depth, index) order of the instances.
//
// The order of one stable sort on the 64-bit key (tile << 32 | depth) is
// produced in two steps: the instances, emitted splat by splat in index
// order, are stably sorted by tile id alone (ceil(log2 tiles) bits, 2 passes
// at a 1008x756 view; 8-byte pairs), and then each tile's run, now in index
// order, is sorted stably by depth inside one workgroup (k_tile_depth_sort,
// at the end of this file).  Sorting the depth per tile in LDS replaces a
// global depth sort of all splats (4 passes of 3 launches each).
//
// Each pass is reduce-then-scan: per-block digit histograms, a per-digit
// scan across blocks, then a scatter in which every block ranks its
// 1024 or 2048 keys stably with wavefront ballots (one ballot per digit bit on
// wave64), sorts them locally in LDS and writes them out digit run by digit
// run, so global stores are contiguous within each run.  The element count
// may live in device memory (the instance count), in which case the grid is
// sized by capacity and blocks past the count exit at once: no host
// synchronisation.  The instance emission writes the first pass's
// histograms of the instance sort itself (its blocks are the sort's blocks),
// which saves that pass's histogram launch.
#include <type_traits>

#include "block_ops.h"
#include "gsp_internal.h"

namespace gsp {

struct SortPass {
    const uint32_t *keys_in;
    const uint32_t *vals_in;
    uint32_t *keys_out;
    uint32_t *vals_out;
    uint32_t *hist;        // [bins][nblk]
    uint32_t *digit_tot;   // [bins]
    const uint32_t *count_ptr;  // element count in device memory, or null
    uint32_t count_val;         // element count when count_ptr is null
    int nblk;
    int shift;
    uint32_t mask;     // digit mask of this pass (at most kSortBins - 1)
    int vbits;         // packed items: the value's bits below the key
};

// Item layout of a pass: a key and a value array (kPairs); one word per
// item, the key above the value's vbits bits (kPacked, when the tile bits
// and the value bits fit 32 between them); or packed items in and the two
// arrays out (kUnpack, the last pass of a packed sort).
enum SortMode { kPairs = 0, kPacked = 1, kUnpack = 2 };

__device__ __forceinline__ uint32_t sort_count(const SortPass &a) {
    return a.count_ptr ? *a.count_ptr : a.count_val;
}

template <int R>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(SortPass a) {
    constexpr int kItems = kSortThreads * R;
    __shared__ uint32_t h[kSortBins];
    const int t = threadIdx.x;
    h[t] = 0;
    __syncthreads();
    const uint32_t M = sort_count(a);
    const size_t base = (size_t)blockIdx.x * kItems;
    if (base < M) {
#pragma unroll 4
        for (int r = 0; r < R; r++) {
            const size_t k = base + (size_t)r * kSortThreads + t;
            if (k < M) atomicAdd(&h[(a.keys_in[k] >> a.shift) & a.mask], 1u);
        }
    }
    __syncthreads();
    if ((uint32_t)t <= a.mask) a.hist[(size_t)t * a.nblk + blockIdx.x] = h[t];   // rows of used digits
}

// One block per digit: exclusive scan of that digit's counts across blocks
// (a row of up to tens of thousands of counts for the instance sort of a
// multi-view call).  The row is scanned in chunks of 4 x 1024 counts: each
// thread loads four consecutive counts of the chunk (the wave's loads cover
// 1 KB contiguously), the block scans the per-thread sums, and the running
// total carries from chunk to chunk.
constexpr int kSortScanThreads = 1024;
constexpr int kSortScanChunk = 4 * kSortScanThreads;

__global__ __launch_bounds__(kSortScanThreads) void k_sort_scan(SortPass a) {
    __shared__ uint32_t scratch[kSortScanThreads / kWave];
    const int t = threadIdx.x;
    uint32_t *row = a.hist + (size_t)blockIdx.x * a.nblk;
    uint32_t carry = 0;
    for (int c0 = 0; c0 < a.nblk; c0 += kSortScanChunk) {
        const int k0 = c0 + 4 * t;
        uint32_t x[4];
#pragma unroll
        for (int j = 0; j < 4; j++) x[j] = k0 + j < a.nblk ? row[k0 + j] : 0u;
        const uint32_t local = x[0] + x[1] + x[2] + x[3];
        uint32_t total;
        uint32_t off = carry + block_exclusive_scan<uint32_t, kSortScanThreads>(local, scratch, &total);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (k0 + j < a.nblk) row[k0 + j] = off;
            off += x[j];
        }
        carry += total;
    }
    if (t == 0) a.digit_tot[blockIdx.x] = carry;
}

template <int R, int MODE>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(SortPass a) {
    constexpr int NW = kSortThreads / kWave;
    constexpr int kItems = kSortThreads * R;
    __shared__ uint32_t skeys[kItems];
    __shared__ uint32_t svals[MODE == kPairs ? kItems : 1];
    __shared__ uint32_t dstart[kSortBins];
    __shared__ uint32_t gbase[kSortBins];
    __shared__ uint32_t run[kSortBins];
    __shared__ uint32_t wcnt[NW][kSortBins];
    __shared__ uint32_t wpre[NW][kSortBins];
    __shared__ uint32_t scratch[kSortThreads / kWave];

    const uint32_t M = sort_count(a);
    const size_t base = (size_t)blockIdx.x * kItems;
    if (base >= M) return;
    const int cnt = (int)min((size_t)kItems, (size_t)M - base);
    const int t = threadIdx.x;
    const int lane = t & (kWave - 1);
    const int w = t / kWave;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;

    uint32_t key[R], val[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int k = r * kSortThreads + t;
        key[r] = k < cnt ? a.keys_in[base + k] : 0u;
        val[r] = MODE == kPairs && k < cnt ? a.vals_in[base + k] : 0u;
    }

    // local histogram -> local digit starts
    run[t] = 0;
#pragma unroll
    for (int w2 = 0; w2 < NW; w2++) wcnt[w2][t] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (r * kSortThreads + t < cnt) atomicAdd(&run[(key[r] >> a.shift) & a.mask], 1u);
    }
    __syncthreads();
    uint32_t tot;
    const uint32_t excl = block_exclusive_scan<uint32_t, kSortThreads>(run[t], scratch, &tot);
    // rows and totals exist for the pass's digits only (mask + 1 of them)
    const bool used = (uint32_t)t <= a.mask;
    const uint32_t digit_total = used ? a.digit_tot[t] : 0u;
    const uint32_t before = used ? a.hist[(size_t)t * a.nblk + blockIdx.x] : 0u;
    const uint32_t dex = block_exclusive_scan<uint32_t, kSortThreads>(digit_total, scratch, &tot);
    dstart[t] = excl;
    run[t] = excl;
    gbase[t] = dex + before;
    __syncthreads();

    // stable ranking, round by round, wave by wave, lane by lane
#pragma unroll 1
    for (int r = 0; r < R; r++) {
        const bool valid = r * kSortThreads + t < cnt;
        const uint32_t d = (key[r] >> a.shift) & a.mask;
        unsigned long long peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kSortBits; b++) {
            if (!((a.mask >> b) & 1u)) break;   // the pass's digit bits only
            const bool bit = (d >> b) & 1u;
            const unsigned long long m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        if (!valid) peers = 0;
        const uint32_t rank = __popcll(peers & lt_mask);
        if (valid && (peers & lt_mask) == 0) wcnt[w][d] = __popcll(peers);
        __syncthreads();
        {
            uint32_t acc = run[t];
#pragma unroll
            for (int w2 = 0; w2 < NW; w2++) {
                const uint32_t c = wcnt[w2][t];
                wcnt[w2][t] = 0;
                wpre[w2][t] = acc;
                acc += c;
            }
            run[t] = acc;
        }
        __syncthreads();
        if (valid) {
            const uint32_t pos = wpre[w][d] + rank;
            skeys[pos] = key[r];
            if (MODE == kPairs) svals[pos] = val[r];
        }
    }
    __syncthreads();

    for (int i = t; i < cnt; i += kSortThreads) {
        const uint32_t k = skeys[i];
        const uint32_t d = (k >> a.shift) & a.mask;
        const size_t dst = (size_t)gbase[d] + (uint32_t)(i - dstart[d]);
        if (MODE == kPairs) {
            a.keys_out[dst] = k;
            a.vals_out[dst] = svals[i];
        } else if (MODE == kPacked) {
            a.keys_out[dst] = k;
        } else {
            a.keys_out[dst] = k >> a.vbits;
            a.vals_out[dst] = k & ((1u << a.vbits) - 1u);
        }
    }
}

// vbits > 0: the input is packed (k0 only) and the passes before the last
// keep it packed; the last pass writes keys and values.
template <int R>
static int launch_sort_pairs(uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1, uint32_t *hist,
                             uint32_t *digit_tot, const uint32_t *count_ptr, uint32_t count_val,
                             int64_t max_count, int bits, bool hist0_given, int vbits, hipStream_t s,
                             hipError_t *err) {
    constexpr int kItems = kSortThreads * R;
    SortPass a;
    a.hist = hist;
    a.digit_tot = digit_tot;
    a.count_ptr = count_ptr;
    a.count_val = count_val;
    a.nblk = (int)((max_count + kItems - 1) / kItems);
    *err = hipSuccess;
    const int passes = sort_passes(bits);
    const int pbits = digit_bits(bits);
    a.mask = (1u << pbits) - 1u;
    if (a.nblk == 0) return passes;
    for (int p = 0; p < passes; p++) {
        a.keys_in = (p & 1) ? k1 : k0;
        a.vals_in = (p & 1) ? v1 : v0;
        a.keys_out = (p & 1) ? k0 : k1;
        a.vals_out = (p & 1) ? v0 : v1;
        a.shift = vbits + p * pbits;
        a.vbits = vbits;
        if (p > 0 || !hist0_given)
            hipLaunchKernelGGL(k_sort_hist<R>, dim3(a.nblk), dim3(kSortThreads), 0, s, a);
        hipLaunchKernelGGL(k_sort_scan, dim3(a.mask + 1), dim3(kSortScanThreads), 0, s, a);
        if (vbits == 0)
            hipLaunchKernelGGL((k_sort_scatter<R, kPairs>), dim3(a.nblk), dim3(kSortThreads), 0, s, a);
        else if (p < passes - 1)
            hipLaunchKernelGGL((k_sort_scatter<R, kPacked>), dim3(a.nblk), dim3(kSortThreads), 0, s, a);
        else
            hipLaunchKernelGGL((k_sort_scatter<R, kUnpack>), dim3(a.nblk), dim3(kSortThreads), 0, s, a);
        *err = hipGetLastError();
        if (*err != hipSuccess) return passes;
    }
    return passes;
}

hipError_t launch_tile_sort(const Layout &L, char *ws, hipStream_t s) {
    hipError_t e;
    auto run = [&](auto rounds) {
        launch_sort_pairs<decltype(rounds)::value>(
            region<uint32_t>(ws, L.keys0), region<uint32_t>(ws, L.vals0), region<uint32_t>(ws, L.keys1),
            region<uint32_t>(ws, L.vals1), region<uint32_t>(ws, L.hist), region<uint32_t>(ws, L.digit_tot),
            region<uint32_t>(ws, L.counters) + kCntMEff, 0u, L.cap, L.tile_bits, true, L.sort_vbits, s,
            &e);
    };
    if (L.sort_items == kSortThreads * kSortRoundsLarge)
        run(std::integral_constant<int, kSortRoundsLarge>{});
    else
        run(std::integral_constant<int, kSortRoundsSmall>{});
    return e;
}


// ---------------------------------------------------------------------------
// Depth order inside each tile.  The instances leave the tile sort grouped by
// tile, each tile's run in index order (they are emitted splat by splat in
// index order and the tile sort is stable).  Each tile's run is then sorted
// stably by the splat's depth key (the float32 bits of its camera-frame z):
// equal depths keep index order, so every run ends in (depth, index) order,
// which is the order of a stable sort of all instances on the 64-bit key
// (tile << 32 | depth).  Only the values (view * n + i) move.
//
// A workgroup sorts a run in LDS by buckets.  The keys are taken relative to
// the run's smallest, and their top bits choose one of CAP buckets; where some
// bucket is crowded (a wall seen in the tile: most depths within a percent),
// every bucket is cut into as many as it has entries, by the key's next bits,
// so that any one cluster is spread as well.  The entries go to their buckets
// in any order, and each finds its place by comparing itself with the others
// of its bucket by (depth, value), which is exact.  A run that stays crowded
// (hundreds of equal depths), or one that does not fit, is sorted in global
// memory by a stable radix sort.
//
// Bound by latency (loads, then some eight steps through LDS with a barrier
// each).  An LSD radix sort in one wavefront's LDS took some 25 LDS operations
// per entry in a chain of ranking rounds; this takes about 10, none waiting for
// another, and a workgroup of four or eight wavefronts shares a run: 23.2 ->
// 15.8 us at 1.5M instances in 3024 lists of 500 (pose step, 1008 x 756; 4.5 us
// more where the kernel of the longer runs finds none), 168 -> 99 + 4.6 us at
// 15.4M in 12096 lists of 1100-1800 (joint step), 79 -> 15.3 + 24.3 us for a
// room with lists of up to 2400, and 706 -> 110 + 118 us for 22M in lists of up
// to 6700 (eight views of three sizes), whose longer half one wavefront each
// had sorted in global memory.
constexpr int kTdCrowd = 12;          // entries of a bucket that are still just compared
constexpr int kTdCrowdMax = 64;       // ... after the buckets were cut
// radix sort in global memory
constexpr int kTdBits = 8, kTdBins = 1 << kTdBits, kTdPasses = 4;

struct TileDepthArgs {
    const uint2 *ranges;
    const uint32_t *order;      // launch order of the tiles, longest first
    const uint32_t *depth;      // [vn] depth key of each view-Gaussian
    uint32_t *keys;             // sorted tile ids (scratch, then restored)
    uint32_t *vals;             // sorted values, put in depth order per tile in place
    uint32_t *akeys, *avals;    // [cap] the tile sort's other buffers (scratch)
    const uint32_t *counters;
    int short_cap;              // longest run of the kernel over all tiles
};

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, off, kWave));
    return v;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, kWave));
    return v;
}

// LDS of a workgroup of THREADS threads, ROUNDS entries each at most.
template <int THREADS, int ROUNDS>
struct TdShared {
    static constexpr int kCap = THREADS * ROUNDS, kWaves = THREADS / kWave;
    union {
        struct {
            uint32_t item[kCap];                      // (key bits below the bucket's, position)
            __align__(16) uint32_t bucket[kCap];      // counts, starts, ends
        };
        struct {                                      // radix sort in global memory
            unsigned long long msk[kWaves][kTdBins];  // lanes of a round by digit
            uint32_t run[kWaves][kTdBins];            // digit counts, then starts
            uint32_t hist[kTdPasses][kTdBins];
        };
    };
    uint32_t part[2 * kWaves];
};

// The block's smallest lo and largest hi.  (Here and below t is threadIdx.x,
// made opaque once per run where a workgroup sorts several: nothing derived
// from it then stays in registers from run to run.)
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_reduce(TdShared<THREADS, ROUNDS> &sh, int t, uint32_t &lo, uint32_t &hi) {
    const int w = t / kWave;
    lo = wave_min_u32(lo);
    hi = wave_max_u32(hi);
    if (t % kWave == 0) {
        sh.part[2 * w] = lo;
        sh.part[2 * w + 1] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < THREADS / kWave; v++) {
        lo = min(lo, sh.part[2 * v]);
        hi = max(hi, sh.part[2 * v + 1]);
    }
}

// Bucket counts -> exclusive starts, in place; returns the largest count.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ uint32_t td_scan(TdShared<THREADS, ROUNDS> &sh, int t) {
    constexpr int kVecs = ROUNDS / 4;
    uint4 *const b = reinterpret_cast<uint4 *>(sh.bucket) + kVecs * t;
    uint4 c[kVecs];
    uint32_t big = 0, s = 0;
#pragma unroll
    for (int j = 0; j < kVecs; j++) {
        c[j] = b[j];
        big = max(big, max(max(c[j].x, c[j].y), max(c[j].z, c[j].w)));
        s += c[j].x + c[j].y + c[j].z + c[j].w;
    }
    const uint32_t inc = wave_inclusive_scan(s);
    big = wave_max_u32(big);
    const int w = t / kWave;
    if (t % kWave == kWave - 1) {
        sh.part[2 * w] = inc;
        sh.part[2 * w + 1] = big;
    }
    __syncthreads();
    uint32_t e = inc - s;
#pragma unroll
    for (int v = 0; v < THREADS / kWave; v++) {
        e += v < w ? sh.part[2 * v] : 0u;
        big = max(big, sh.part[2 * v + 1]);
    }
#pragma unroll
    for (int j = 0; j < kVecs; j++) {
        b[j] = make_uint4(e, e + c[j].x, e + c[j].x + c[j].y, e + c[j].x + c[j].y + c[j].z);
        e += c[j].x + c[j].y + c[j].z + c[j].w;
    }
    __syncthreads();
    return big;
}

template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_zero(TdShared<THREADS, ROUNDS> &sh, int t) {
#pragma unroll
    for (int j = 0; j < ROUNDS / 4; j++)
        reinterpret_cast<uint4 *>(sh.bucket)[j * THREADS + t] = make_uint4(0, 0, 0, 0);
}

// Sorts a run of at most THREADS ROUNDS entries in LDS.  Returns false, with
// nothing changed, if a bucket stays crowded.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ bool td_sort_lds(const TileDepthArgs &a, TdShared<THREADS, ROUNDS> &sh,
                                            int t, uint32_t *vf, int L) {
    constexpr uint32_t kCap = TdShared<THREADS, ROUNDS>::kCap;
    constexpr int kLog = 31 - __builtin_clz(kCap);   // bits of a bucket, and of a position in the run
    static_assert(kCap == 1u << kLog, "a power of two");
    // Which entries a thread has is worked out afresh in each phase: the lane
    // masks of all rounds, kept through the function, do not fit the scalar
    // registers.
    auto phase = [&]() { asm volatile("" : "+v"(t)); };
    // (with 16 entries per thread the values are read again at the end: held,
    // they would cost registers spilled to memory)
    constexpr bool kReload = ROUNDS > 8;
    uint32_t key[ROUNDS], val[ROUNDS], bin[ROUNDS];
    auto load_values = [&]() {
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            const int k = r * THREADS + t;
            val[r] = k < L ? vf[k] : 0u;
        }
    };
    load_values();
    td_zero(sh, t);
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            key[r] = a.depth[val[r]];
            kmin = min(kmin, key[r]);
            kmax = max(kmax, key[r]);
        }
    }
    td_reduce(sh, t, kmin, kmax);
    if (kmin == kmax) return true;   // one depth: nothing moves
    // Depths lie between the near plane and infinity, so a relative key has
    // at most 31 bits, and those below the bucket's leave room for a position
    // in an entry's word.
    const int B = 32 - __clz(kmax - kmin), sft = B > kLog ? B - kLog : 0;
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            key[r] -= kmin;
            bin[r] = key[r] >> sft;
            atomicAdd(&sh.bucket[bin[r]], 1u);
            key[r] &= (1u << sft) - 1u;
        }
    }
    __syncthreads();
    if (td_scan(sh, t) > kTdCrowd) {
        // cut every bucket by the key's next bits into as many as it has
        // entries: bucket b's start on, in place of b
        phase();
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            if (r * THREADS + t < L) {
                const uint32_t s = sh.bucket[bin[r]], e = bin[r] + 1 < kCap ? sh.bucket[bin[r] + 1] : (uint32_t)L;
                bin[r] = s + __umulhi(sft > 0 ? key[r] << (32 - sft) : 0u, e - s);
            }
        }
        __syncthreads();
        td_zero(sh, t);
        __syncthreads();
        phase();
#pragma unroll
        for (int r = 0; r < ROUNDS; r++)
            if (r * THREADS + t < L) atomicAdd(&sh.bucket[bin[r]], 1u);
        __syncthreads();
        if (td_scan(sh, t) > kTdCrowdMax) return false;
    }
    // to the buckets, in any order; bucket[b] ends as the end of b
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            key[r] = key[r] << kLog | (uint32_t)(r * THREADS + t);
            sh.item[atomicAdd(&sh.bucket[bin[r]], 1u)] = key[r];
        }
    }
    __syncthreads();
    // bin[r] becomes the entry's place
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            const uint32_t s = bin[r] > 0 ? sh.bucket[bin[r] - 1] : 0u, e = sh.bucket[bin[r]];
            bin[r] = s;
            for (uint32_t j = s; j < e; j++) bin[r] += sh.item[j] < key[r] ? 1u : 0u;
        }
    }
    phase();
    if (kReload) load_values();
    __syncthreads();
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) sh.item[bin[r]] = val[r];
    __syncthreads();
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) vf[r * THREADS + t] = sh.item[r * THREADS + t];
    return true;
}

// Rank of the lane's item among the lanes of its round with the same digit,
// plus run[d], the count of d in earlier rounds.  The lanes with digit d find
// each other through msk[d]: each ORs its lane bit in, then reads the mask
// back (a wavefront's LDS accesses take effect in program order, so every OR
// lands before any read); the lowest of them advances run[d] and clears
// msk[d] for the next round.  msk must be zero on entry and is zero again on
// return.
__device__ __forceinline__ uint32_t td_rank(int lane, bool valid, uint32_t d, uint32_t *run,
                                            unsigned long long *msk) {
    const unsigned long long lt = (1ull << lane) - 1ull;
    if (valid) atomicOr(&msk[d], 1ull << lane);
    const unsigned long long peers = valid ? msk[d] : 0ull;
    const uint32_t below = __popcll(peers & lt);
    const uint32_t base = valid ? run[d] : 0u;
    if (valid && below == 0) {
        run[d] = base + (uint32_t)__popcll(peers);
        msk[d] = 0ull;
    }
    return base + below;
}

// A run in global memory, sorted LSD over 8-bit digits of the relative depth
// keys: the smallest key, then the histograms of every pass from two reads of
// the run (keys gathered), then the passes (skipped where every digit is
// zero), each a stable counting sort: a chunk's items counted per wavefront,
// the counts' starts, then each wavefront's ranks on top of them.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_sort_global(const TileDepthArgs &a, TdShared<THREADS, ROUNDS> &sh,
                                               int t, uint32_t rgx, uint32_t tile, int L) {
    constexpr int kWaves = THREADS / kWave, kSeg = ROUNDS * kWave;
    const int lane = t & (kWave - 1), w = t / kWave;
    uint32_t *const kf = a.keys + rgx, *const vf = a.vals + rgx;
    uint32_t kmin = 0xffffffffu, unused = 0u;
    for (int k = t; k < L; k += THREADS) kmin = min(kmin, a.depth[vf[k]]);
    __syncthreads();
    td_reduce(sh, t, kmin, unused);
    for (int i = t; i < kTdPasses * kTdBins; i += THREADS) (&sh.hist[0][0])[i] = 0u;
    for (int i = lane; i < kTdBins; i += kWave) sh.msk[w][i] = 0ull;
    __syncthreads();
    for (int k = t; k < L; k += THREADS) {
        const uint32_t kk = a.depth[vf[k]] - kmin;
#pragma unroll
        for (int p = 0; p < kTdPasses; p++) atomicAdd(&sh.hist[p][(kk >> (kTdBits * p)) & (kTdBins - 1)], 1u);
    }
    __syncthreads();
    // source of the next pass: (keys gathered | skey, sval), destination (dkey, dval)
    uint32_t *skey = nullptr, *sval = vf, *dkey = a.akeys + rgx, *dval = a.avals + rgx;
    bool kf_used = false;
    for (int p = 0; p < kTdPasses; p++) {
        const int sft = kTdBits * p;
        if (sh.hist[p][0] == (uint32_t)L) continue;   // all zero: nothing moves
        __syncthreads();
        if (w == 0) {   // counts -> starts of the digits, four per lane
            uint32_t *const h = &sh.hist[p][4 * lane];
            const uint32_t c0 = h[0], c1 = h[1], c2 = h[2], c3 = h[3];
            const uint32_t e = wave_inclusive_scan(c0 + c1 + c2 + c3) - (c0 + c1 + c2 + c3);
            h[0] = e;
            h[1] = e + c0;
            h[2] = e + c0 + c1;
            h[3] = e + c0 + c1 + c2;
        }
        auto key_of = [&](int k) { return skey ? skey[k] : a.depth[sval[k]] - kmin; };
        for (int c0 = 0; c0 < L; c0 += THREADS * ROUNDS) {
            const int k0 = c0 + w * kSeg, end = min(L, k0 + kSeg);
            for (int i = lane; i < kTdBins; i += kWave) sh.run[w][i] = 0u;
            __syncthreads();
            for (int k = k0 + lane; k < end; k += kWave)
                atomicAdd(&sh.run[w][(key_of(k) >> sft) & (kTdBins - 1)], 1u);
            __syncthreads();
            for (int d = t; d < kTdBins; d += THREADS) {
                uint32_t e = sh.hist[p][d];
#pragma unroll
                for (int v = 0; v < kWaves; v++) {
                    const uint32_t c = sh.run[v][d];
                    sh.run[v][d] = e;
                    e += c;
                }
                sh.hist[p][d] = e;
            }
            __syncthreads();
#pragma unroll 1
            for (int r0 = k0; r0 < end; r0 += kWave) {
                const int k = r0 + lane;
                const uint32_t key = k < end ? key_of(k) : 0u;
                const uint32_t pos = td_rank(lane, k < end, (key >> sft) & (kTdBins - 1), sh.run[w], sh.msk[w]);
                if (k < end) {
                    dkey[pos] = key;
                    dval[pos] = sval[k];
                }
            }
            __syncthreads();
        }
        kf_used |= dkey == kf;
        uint32_t *const nk = dkey == kf ? a.akeys + rgx : kf;
        uint32_t *const nv = dval == vf ? a.avals + rgx : vf;
        skey = dkey;
        sval = dval;
        dkey = nk;
        dval = nv;
    }
    if (sval != vf)
        for (int k = t; k < L; k += THREADS) vf[k] = sval[k];
    if (kf_used)
        for (int k = t; k < L; k += THREADS) kf[k] = tile;
    __syncthreads();
}

// Workgroup b takes tile b, so that its first load is its range.  An
// overflowing forward emits no instance and leaves every range empty, so
// neither kernel needs an overflow test.
template <int THREADS, int ROUNDS>
__global__ __launch_bounds__(THREADS) void k_tile_depth_sort(TileDepthArgs a) {
    __shared__ TdShared<THREADS, ROUNDS> sh;
    const uint32_t tile = blockIdx.x;
    const uint2 rg = a.ranges[tile];
    const int L = (int)(rg.y - rg.x);
    if (L <= 1 || L > THREADS * ROUNDS) return;
    const int t = threadIdx.x;
    if (!td_sort_lds(a, sh, t, a.vals + rg.x, L)) td_sort_global(a, sh, t, rg.x, tile, L);
}

// The longer runs, at the front of the launch order.
constexpr int kTdLongThreads = 512, kTdLongRounds = 16;
__global__ __launch_bounds__(kTdLongThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_tile_depth_sort_long(TileDepthArgs a) {
    __shared__ TdShared<kTdLongThreads, kTdLongRounds> sh;
    const uint32_t nlong = a.counters[a.short_cap == 1024 ? kCntOver1024 : kCntOver2048];
    for (uint32_t r = blockIdx.x; r < nlong; r += gridDim.x) {
        const uint32_t tile = a.order[r];
        const uint2 rg = a.ranges[tile];
        const int L = (int)(rg.y - rg.x);
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        __syncthreads();
        if (L > kTdLongThreads * kTdLongRounds || !td_sort_lds(a, sh, t, a.vals + rg.x, L))
            td_sort_global(a, sh, t, rg.x, tile, L);
    }
}

hipError_t launch_tile_depth_sort(const Layout &L, char *ws, hipStream_t s) {
    if (L.total_tiles == 0) return hipSuccess;
    TileDepthArgs a;
    const bool odd = sorted_vals(L) == L.vals1;
    a.ranges = region<uint2>(ws, L.ranges);
    a.order = region<uint32_t>(ws, L.tile_order);
    a.depth = region<uint32_t>(ws, L.depth);
    a.keys = region<uint32_t>(ws, sorted_keys(L));
    a.vals = region<uint32_t>(ws, sorted_vals(L));
    a.akeys = region<uint32_t>(ws, odd ? L.keys0 : L.keys1);
    a.avals = region<uint32_t>(ws, odd ? L.vals0 : L.vals1);
    a.counters = region<uint32_t>(ws, L.counters);
    // Lists longer than 1024 on average (at the 1.5x capacity margin) take
    // eight entries per thread, which keep them in this launch; for lists of
    // 500 four per thread measured 15.8 us against 16.3, of 700 42.8 against
    // 45.4 us.  (128 threads of eight: 15.5 and 46.9 us.)
    const bool mid = L.cap > (int64_t)1536 * L.total_tiles;
    a.short_cap = mid ? 2048 : 1024;
    if (mid)
        hipLaunchKernelGGL((k_tile_depth_sort<256, 8>), dim3(L.total_tiles), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((k_tile_depth_sort<256, 4>), dim3(L.total_tiles), dim3(256), 0, s, a);
    // a list holds a splat once at most; two of these workgroups fit a CU
    if (L.n > a.short_cap)
        hipLaunchKernelGGL(k_tile_depth_sort_long, dim3(L.total_tiles < 512 ? L.total_tiles : 512),
                           dim3(kTdLongThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace gsp
