// sort.hip -- the (depth, index) order inside each tile's list.
//
// The binning leaves the instances grouped by tile, each a (depth key, view * n
// + i) pair; each tile's run is put in the order of a stable sort by the
// splat's depth key (the float32 bits of its camera-frame z) of the splats in
// index order, equal depths in index order, which makes the whole the order of
// a stable sort of all instances on the 64-bit key (tile << 32 | depth).  Only
// the values (view * n + i) are written.
//
// A workgroup sorts a run in LDS by buckets.  The keys are taken relative to
// the run's smallest, and their top bits choose one of CAP buckets; where some
// bucket is crowded (a wall seen in the tile: most depths within a percent),
// every bucket is cut into as many as it has entries, by the key's next bits,
// so that any one cluster is spread as well.  The entries go to their buckets
// in any order, and each finds its place by comparing itself with the others
// of its bucket by (depth, value), which is exact.  A run that stays crowded
// with equal depths (more than kTdCrowdMax, as of a wall that faces the camera)
// is ranked by value first, and the ranks cut its buckets: 3225 lists of 760
// entries in three walls take 69 us (19 us where the depths differ), and took 139
// in the global-memory sort.  Crowds of different depths go through a bitonic
// network in LDS, and a run that does not fit is sorted in global memory by a
// stable radix sort over value and depth.
//
// Bound by latency (loads, then some eight steps through LDS with a barrier
// each).  An LSD radix sort in one wavefront's LDS took some 25 LDS operations
// per entry in a chain of ranking rounds; this takes about 10, none waiting for
// another, and a workgroup of four or eight wavefronts shares a run: 23.2 ->
// 13.0 us at 1.5M instances in 3024 lists of 500 (pose step, 1008 x 756; 4.5 us
// more where the kernel of the longer runs finds none), 168 -> 76 + 4.5 us at
// 15.4M in 12096 lists of 1100-1800 (joint step), 79 -> 13.8 + 23 us for a
// room with lists of up to 2400, and 706 -> 87 + 78 us for 22M in lists of up
// to 6700 (eight views of three sizes), whose longer half one wavefront each
// had sorted in global memory.  (The tile ids for inspection are 1 to 9 us of it.)
#include "block_ops.h"
#include "gsp_internal.h"

namespace gsp {

constexpr int kTdCrowd = 12;          // entries of a bucket that are still just compared
constexpr int kTdCrowdMax = 64;       // ... after the buckets were cut
// radix sort in global memory
constexpr int kTdBits = 8, kTdBins = 1 << kTdBits;

struct TileDepthArgs {
    const uint2 *ranges;
    const uint32_t *order;      // launch order of the tiles, longest first
    uint2 *pairs;               // (depth key, value) of the instances, grouped by tile
    uint2 *spare;               // [cap] scratch of the radix sort
    uint32_t *vals;             // the values in (tile, depth, value) order
    uint32_t *keys;             // the tile of each of them
    const uint32_t *counters;
    int short_cap;              // longest run of the kernel over all tiles
};

// LDS of a workgroup of THREADS threads, ROUNDS entries each at most.
template <int THREADS, int ROUNDS>
struct TdShared {
    static constexpr int kCap = THREADS * ROUNDS, kWaves = THREADS / kWave;
    union {
        struct {
            uint32_t item[kCap];                      // (key bits below the bucket's, position)
            __align__(16) uint32_t bucket[kCap];      // counts, starts, ends
        };
        unsigned long long pair[kCap];                // (depth key, value), bitonic network
        struct {                                      // radix sort in global memory
            unsigned long long msk[kWaves][kTdBins];  // lanes of a round by digit
            uint32_t run[kWaves][kTdBins];            // digit counts, then starts
            uint32_t hist[kTdBins];
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
    lo = wave_min(lo);
    hi = wave_max(hi);
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

// Whether the condition holds in some thread of the block (which waits here).
template <int THREADS, int ROUNDS>
__device__ __forceinline__ bool td_any(TdShared<THREADS, ROUNDS> &sh, int t, bool p) {
    const uint32_t any = wave_any(p) ? 1u : 0u;
    if (t % kWave == 0) sh.part[t / kWave] = any;
    __syncthreads();
    uint32_t all = 0u;
#pragma unroll
    for (int v = 0; v < THREADS / kWave; v++) all |= sh.part[v];
    return all != 0u;
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
    big = wave_max(big);
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

// Counts of the entries' bins -> starts of the buckets; returns the largest
// count.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ uint32_t td_buckets(TdShared<THREADS, ROUNDS> &sh, int &t, int L,
                                               const uint32_t (&bin)[ROUNDS]) {
    __syncthreads();
    td_zero(sh, t);
    __syncthreads();
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) atomicAdd(&sh.bucket[bin[r]], 1u);
    __syncthreads();
    return td_scan(sh, t);
}

// Start and number of entries of bucket b, from the starts.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_bucket(const TdShared<THREADS, ROUNDS> &sh, int L, uint32_t b, uint32_t &s,
                                          uint32_t &m) {
    s = sh.bucket[b];
    m = (b + 1 < (uint32_t)TdShared<THREADS, ROUNDS>::kCap ? sh.bucket[b + 1] : (uint32_t)L) - s;
}

// The entries' places: each goes to its bucket, in any order, with a word that
// none shares (key), and counts the words below its own there.  bin becomes the
// place.  (bucket[b] ends as the end of b.)
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_places(TdShared<THREADS, ROUNDS> &sh, int &t, int L, const uint32_t (&key)[ROUNDS],
                                          uint32_t (&bin)[ROUNDS]) {
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) sh.item[atomicAdd(&sh.bucket[bin[r]], 1u)] = key[r];
    __syncthreads();
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            const uint32_t s = bin[r] > 0 ? sh.bucket[bin[r] - 1] : 0u, e = sh.bucket[bin[r]];
            bin[r] = s;
            for (uint32_t j = s; j < e; j++) bin[r] += sh.item[j] < key[r] ? 1u : 0u;
        }
    }
    __syncthreads();
}

// A run that td_sort_buckets left with crowded buckets (in `bin`, and their starts
// in LDS; with 16 entries per thread they are formed anew): equal depths.  The
// entries' ranks by value come from buckets of the values, cut like those of the
// depths; the values of a run differ, so no more than the square root of 2^(bits
// of the values' range - kLog) of them meet in a bucket (32 for a million splats
// and 1024 entries).  A bucket of the depths whose m entries are of one depth is
// then cut by rank, which leaves at most L / m + 1 of them together.  Returns
// false, with nothing changed, if a crowded bucket holds different depths.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ bool td_sort_ties(const TileDepthArgs &a, TdShared<THREADS, ROUNDS> &sh, int t,
                                             uint32_t rgx, int L, uint32_t kmin, int sft, uint32_t (&bin)[ROUNDS]) {
    constexpr int kLog = 31 - __builtin_clz((uint32_t)TdShared<THREADS, ROUNDS>::kCap);
    constexpr bool kMany = ROUNDS > 8;
    const uint2 *const run = a.pairs + rgx;
    uint32_t *const aside = reinterpret_cast<uint32_t *>(a.spare + rgx);
    uint32_t key[ROUNDS], val[ROUNDS];
    auto phase = [&]() { asm volatile("" : "+v"(t)); };
    // (with 16 entries per thread, no more than four entries' loads in flight)
    auto pace = [&](int r) __attribute__((always_inline)) {
        if (kMany && r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    };
    auto load_keys = [&](int bits) __attribute__((always_inline)) {   // the lowest bits
        phase();
#pragma unroll
        for (int r = 0; r < ROUNDS; r++)
            key[r] = r * THREADS + t < L ? (run[r * THREADS + t].x - kmin) & ((1u << bits) - 1u) : 0u;
    };
    if constexpr (kMany) {   // the buckets of the depths, cut, once more
        load_keys(31);
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            bin[r] = key[r] >> sft;
            key[r] &= (1u << sft) - 1u;
        }
        td_buckets(sh, t, L, bin);
        phase();
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            if (r * THREADS + t < L) {
                uint32_t s, m;
                td_bucket(sh, L, bin[r], s, m);
                bin[r] = s + __umulhi(sft > 0 ? key[r] << (32 - sft) : 0u, m);
            }
            pace(r);
        }
        td_buckets(sh, t, L, bin);
    } else {
        load_keys(sft);
    }
    // a bucket's word: some key of it, or ~0 (no key) if it has others too (bit
    // 31 of an entry's bin: its key is not the word, then: the word is a key)
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) sh.item[bin[r]] = key[r];
    __syncthreads();
    bool differ = false;
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            uint32_t s, m;
            td_bucket(sh, L, bin[r], s, m);
            const bool other = sh.item[bin[r]] != key[r];
            differ |= other && m > kTdCrowdMax;
            bin[r] |= other ? 0x80000000u : 0u;
        }
        pace(r);
    }
    if (td_any(sh, t, differ)) return false;
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L && (bin[r] >> 31) != 0u) sh.item[bin[r] &= 0x7fffffffu] = 0xffffffffu;
    __syncthreads();
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) bin[r] |= sh.item[bin[r]] != 0xffffffffu ? 0x80000000u : 0u;
    if constexpr (kMany) {   // put aside: they would not fit the registers beside the values
        phase();
#pragma unroll
        for (int r = 0; r < ROUNDS; r++)
            if (r * THREADS + t < L) aside[r * THREADS + t] = bin[r];
    }
    // ranks by value
    uint32_t vmin = 0xffffffffu, vmax = 0u;
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        val[r] = r * THREADS + t < L ? run[r * THREADS + t].y : 0u;
        if (r * THREADS + t < L) {
            vmin = min(vmin, val[r]);
            vmax = max(vmax, val[r]);
        }
    }
    td_reduce(sh, t, vmin, vmax);
    const int vb = vmax > vmin ? 32 - __clz(vmax - vmin) : 0, vsft = vb > kLog ? vb - kLog : 0;
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        val[r] -= vmin;
        key[r] = val[r] >> vsft;
    }
    if (td_buckets(sh, t, L, key) > kTdCrowd) {
        phase();
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            if (r * THREADS + t < L) {
                uint32_t s, m;
                td_bucket(sh, L, key[r], s, m);
                key[r] = s + __umulhi(vsft > 0 ? val[r] << (32 - vsft) : 0u, m);
            }
            pace(r);
        }
        td_buckets(sh, t, L, key);
    }
    td_places(sh, t, L, val, key);
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) val[r] = key[r];   // the rank
    // the buckets of the depths again, those of one depth cut by rank
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if constexpr (kMany) bin[r] = r * THREADS + t < L ? aside[r * THREADS + t] : 0u;
        key[r] = bin[r] & 0x7fffffffu;
    }
    td_buckets(sh, t, L, key);
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            uint32_t s, m;
            td_bucket(sh, L, key[r], s, m);
            bin[r] = s + (bin[r] >> 31 ? val[r] * m / (uint32_t)L : 0u);
        }
        pace(r);
    }
    td_buckets(sh, t, L, bin);
    load_keys(sft);
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) key[r] = key[r] << kLog | val[r];
    td_places(sh, t, L, key, bin);
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) a.vals[rgx + bin[r]] = run[r * THREADS + t].y;
    return true;
}

// Sorts a run of at most THREADS ROUNDS entries in LDS.  Returns false, with
// nothing changed, if a bucket stays crowded.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ bool td_sort_buckets(const TileDepthArgs &a, TdShared<THREADS, ROUNDS> &sh,
                                                int t, uint32_t rgx, int L, uint32_t &kmin, int &sft,
                                                uint32_t (&bin)[ROUNDS]) {
    constexpr uint32_t kCap = TdShared<THREADS, ROUNDS>::kCap;
    constexpr int kLog = 31 - __builtin_clz(kCap);   // bits of a bucket, and of a position in the run
    static_assert(kCap == 1u << kLog, "a power of two");
    // Which entries a thread has is worked out afresh in each phase: the lane
    // masks of all rounds, kept through the function, do not fit the scalar
    // registers.
    auto phase = [&]() { asm volatile("" : "+v"(t)); };
    const uint2 *const run = a.pairs + rgx;
    // (with 16 entries per thread the values are read again at the end: held,
    // they would cost registers spilled to memory)
    constexpr bool kReload = ROUNDS > 8;
    uint32_t key[ROUNDS], val[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        const int k = r * THREADS + t;
        const uint2 p = k < L ? run[k] : make_uint2(0u, 0u);
        key[r] = p.x;
        val[r] = p.y;
    }
    td_zero(sh, t);
    uint32_t kmax = 0u;
    kmin = 0xffffffffu;
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        if (r * THREADS + t < L) {
            kmin = min(kmin, key[r]);
            kmax = max(kmax, key[r]);
        }
    }
    td_reduce(sh, t, kmin, kmax);
    // Depths lie between the near plane and infinity, so a relative key has
    // at most 31 bits, and those below the bucket's leave room for a position
    // in an entry's word.
    const int B = kmax > kmin ? 32 - __clz(kmax - kmin) : 0;
    sft = B > kLog ? B - kLog : 0;
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
        if (td_buckets(sh, t, L, bin) > kTdCrowdMax) return false;
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
            for (uint32_t j = s; j < e; j++) {
                const uint32_t other = sh.item[j];
                bool less = other < key[r];
                // equal depths: the splats' order (chunks of the binning are in
                // index order, the entries of one are not)
                if ((other ^ key[r]) - 1u < kCap - 1u)
                    less = run[other & (kCap - 1u)].y < run[key[r] & (kCap - 1u)].y;
                bin[r] += less ? 1u : 0u;
            }
        }
    }
    phase();
    if (kReload) {
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) val[r] = r * THREADS + t < L ? run[r * THREADS + t].y : 0u;
    }
    __syncthreads();
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) sh.item[bin[r]] = val[r];
    __syncthreads();
    phase();
#pragma unroll
    for (int r = 0; r < ROUNDS; r++)
        if (r * THREADS + t < L) a.vals[rgx + r * THREADS + t] = sh.item[r * THREADS + t];
    return true;
}

// Sorts a run of 2 to THREADS ROUNDS entries in LDS, whatever its keys: a bitonic
// network over the (depth key, value) pairs, padded to a power of two.  At
// distances of 64 and less a wavefront's comparisons take 128 neighbouring entries
// of its own, so that between two such steps a wave waits for no other.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_sort_bitonic(const TileDepthArgs &a, TdShared<THREADS, ROUNDS> &sh,
                                                int t, uint32_t rgx, int L) {
    const uint2 *const run = a.pairs + rgx;
    const int P = 1 << (32 - __clz(L - 1));
    for (int k = t; k < P; k += THREADS) {
        const uint2 p = k < L ? run[k] : make_uint2(0xffffffffu, 0xffffffffu);
        sh.pair[k] = (unsigned long long)p.x << 32 | p.y;
    }
    __syncthreads();
#pragma unroll 1
    for (int size = 2; size <= P; size *= 2) {
#pragma unroll 1
        for (int d = size / 2; d > 0; d /= 2) {
            for (int i = t; i < P / 2; i += THREADS) {
                const int k = 2 * i - (i & (d - 1));
                const unsigned long long x = sh.pair[k], y = sh.pair[k + d];
                if ((x > y) == ((k & size) == 0)) {
                    sh.pair[k] = y;
                    sh.pair[k + d] = x;
                }
            }
            // (the next step's distance: d / 2, or size behind the last)
            if (d > kWave || (d == 1 && size > kWave)) __syncthreads();
            else wave_sync();
        }
    }
    __syncthreads();
    for (int k = t; k < L; k += THREADS) a.vals[rgx + k] = (uint32_t)sh.pair[k];
}

// Sorts a run of at most THREADS ROUNDS entries in LDS.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_sort_lds(const TileDepthArgs &a, TdShared<THREADS, ROUNDS> &sh, int t,
                                            uint32_t rgx, int L) {
    uint32_t kmin;
    int sft;
    // (where the ties are put in buckets anew, their bins are other registers:
    // kept from here, they would be spilled from run to run)
    uint32_t bin[ROUNDS], ties[ROUNDS];
    if (!td_sort_buckets(a, sh, t, rgx, L, kmin, sft, bin) &&
        !td_sort_ties(a, sh, t, rgx, L, kmin, sft, ROUNDS > 8 ? ties : bin))
        td_sort_bitonic(a, sh, t, rgx, L);
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

// A run in global memory, sorted LSD over the 8-bit digits of the values and
// then of the depth keys, both relative to the run's smallest.  A pass is a
// stable counting sort: the digits' counts (nothing moves if all are zero) and
// starts, then, a chunk at a time, the counts of each wavefront's items, their
// starts, and each wavefront's ranks on top of them.
template <int THREADS, int ROUNDS>
__device__ __forceinline__ void td_sort_global(const TileDepthArgs &a, TdShared<THREADS, ROUNDS> &sh,
                                               int t, uint32_t rgx, int L) {
    constexpr int kWaves = THREADS / kWave, kSeg = ROUNDS * kWave, kPasses = 2 * 32 / kTdBits;
    const int lane = t & (kWave - 1), w = t / kWave;
    uint2 *src = a.pairs + rgx, *dst = a.spare + rgx;
    uint32_t kmin = 0xffffffffu, vmin = 0xffffffffu, unused = 0u;
    for (int k = t; k < L; k += THREADS) {
        const uint2 p = src[k];
        kmin = min(kmin, p.x);
        vmin = min(vmin, p.y);
    }
    __syncthreads();
    td_reduce(sh, t, kmin, unused);
    __syncthreads();
    td_reduce(sh, t, vmin, unused);
    for (int i = lane; i < kTdBins; i += kWave) sh.msk[w][i] = 0ull;
    for (int p = 0; p < kPasses; p++) {
        const bool by_value = p < kPasses / 2;
        const int sft = kTdBits * (by_value ? p : p - kPasses / 2);
        auto digit = [&](const uint2 &q) { return ((by_value ? q.y - vmin : q.x - kmin) >> sft) & (kTdBins - 1); };
        for (int i = t; i < kTdBins; i += THREADS) sh.hist[i] = 0u;
        __syncthreads();
        for (int k = t; k < L; k += THREADS) atomicAdd(&sh.hist[digit(src[k])], 1u);
        __syncthreads();
        if (sh.hist[0] == (uint32_t)L) {
            __syncthreads();
            continue;
        }
        __syncthreads();
        if (w == 0) {   // counts -> starts of the digits, four per lane
            uint32_t *const h = &sh.hist[4 * lane];
            const uint32_t c0 = h[0], c1 = h[1], c2 = h[2], c3 = h[3];
            const uint32_t e = wave_inclusive_scan(c0 + c1 + c2 + c3) - (c0 + c1 + c2 + c3);
            h[0] = e;
            h[1] = e + c0;
            h[2] = e + c0 + c1;
            h[3] = e + c0 + c1 + c2;
        }
        for (int c0 = 0; c0 < L; c0 += THREADS * ROUNDS) {
            const int k0 = c0 + w * kSeg, end = min(L, k0 + kSeg);
            for (int i = lane; i < kTdBins; i += kWave) sh.run[w][i] = 0u;
            __syncthreads();
            for (int k = k0 + lane; k < end; k += kWave) atomicAdd(&sh.run[w][digit(src[k])], 1u);
            __syncthreads();
            for (int d = t; d < kTdBins; d += THREADS) {
                uint32_t e = sh.hist[d];
#pragma unroll
                for (int v = 0; v < kWaves; v++) {
                    const uint32_t c = sh.run[v][d];
                    sh.run[v][d] = e;
                    e += c;
                }
                sh.hist[d] = e;
            }
            __syncthreads();
#pragma unroll 1
            for (int r0 = k0; r0 < end; r0 += kWave) {
                const int k = r0 + lane;
                const uint2 q = k < end ? src[k] : make_uint2(0u, 0u);
                const uint32_t pos = td_rank(lane, k < end, digit(q), sh.run[w], sh.msk[w]);
                if (k < end) dst[pos] = q;
            }
            __syncthreads();
        }
        uint2 *const other = src;
        src = dst;
        dst = other;
    }
    for (int k = t; k < L; k += THREADS) a.vals[rgx + k] = src[k].y;
    __syncthreads();
}

// The tile of each entry of a run: for inspection alone (4 bytes per instance, 10 of
// 83 us at 15.4M of them), but written here, where every forward of a stream or a
// graph has it in its order.
template <int THREADS>
__device__ __forceinline__ void td_keys(const TileDepthArgs &a, uint32_t tile, const uint2 &rg) {
    for (uint32_t k = rg.x + threadIdx.x; k < rg.y; k += THREADS) a.keys[k] = tile;
}

// Workgroup b takes tile b, so that its first load is its range.  An
// overflowing forward emits no instance and leaves every range empty, so
// neither kernel needs an overflow test.
template <int THREADS, int ROUNDS>
__global__ __launch_bounds__(THREADS) void k_tile_depth_sort(TileDepthArgs a) {
    __shared__ TdShared<THREADS, ROUNDS> sh;
    const uint2 rg = a.ranges[blockIdx.x];
    const int L = (int)(rg.y - rg.x);
    if (L < 1 || L > THREADS * ROUNDS) return;
    const int t = threadIdx.x;
    td_sort_lds(a, sh, t, rg.x, L);
    td_keys<THREADS>(a, blockIdx.x, rg);
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
        if (L > kTdLongThreads * kTdLongRounds) td_sort_global(a, sh, t, rg.x, L);
        else td_sort_lds(a, sh, t, rg.x, L);
        td_keys<kTdLongThreads>(a, tile, rg);
    }
}

hipError_t launch_tile_depth_sort(const Layout &L, char *ws, hipStream_t s) {
    if (L.total_tiles == 0) return hipSuccess;
    TileDepthArgs a;
    a.ranges = region<uint2>(ws, L.ranges);
    a.order = region<uint32_t>(ws, L.tile_order);
    a.pairs = region<uint2>(ws, L.pairs);
    // the gradient slots (36 bytes per instance) are the backward's
    a.spare = region<uint2>(ws, L.slots);
    a.vals = region<uint32_t>(ws, L.vals);
    a.keys = region<uint32_t>(ws, L.keys);
    a.counters = region<uint32_t>(ws, L.counters);
    // Eight entries per thread keep lists of up to 2048 in this launch, where four
    // leave those above 1024 to the long kernel: 1.1 times four's time for lists of
    // 450 to 500 on average, 1.02 to 1.06 for 600 to 750, 1.01 for 800 and 900 in a
    // few even tiles, but 0.75 for 860, 0.66 to 0.79 for 940 to 990 and 0.4 to 0.5
    // above 1000, as the first lists pass 1024.  The instances' number is not known
    // here; the line is at 850 for a capacity of 1.5 times as many.
    const bool mid = L.cap > (int64_t)1280 * L.total_tiles;
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
