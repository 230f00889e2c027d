// block_ops.h -- wavefront (64 lanes) and block reductions and scans used by
// the gfx950 kernels.  Lanes exchange values in the VALU (v_permlane32_swap,
// v_permlane16_swap and DPP moves), each step a few cycles instead of an LDS
// round trip (ds_bpermute); block-level steps go through LDS.  All lanes of the
// wavefront must be active.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gsp {

constexpr int kWave = 64;

// Wave-wide vote on a lane predicate, straight from the compare's lane mask
// (no round trip of the predicate through a vector register).
__device__ __forceinline__ bool wave_any(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// Orders a wavefront's LDS accesses before this point against those after it
// for the compiler (the hardware executes them in program order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A 4- or 8-byte value through a 32-bit lane exchange.
template <typename T, typename F>
__device__ __forceinline__ T by_words(T v, F exchange) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "whole registers");
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, exchange(__builtin_bit_cast(uint32_t, v)));
    } else {
        const uint64_t x = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = exchange((uint32_t)x), hi = exchange((uint32_t)(x >> 32));
        return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
    }
}

// v of one lane (the same in all lanes).
template <typename T>
__device__ __forceinline__ T wave_lane(T v, int lane) {
    return by_words(v, [=](uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, lane); });
}

// v moved by a DPP control within the rows of 16 lanes; lanes without a source
// (and rows not in ROWS) get zero.
template <int CTRL, int ROWS = 0xF, typename T>
__device__ __forceinline__ T dpp_move(T v) {
    return by_words(v, [](uint32_t x) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, true);
    });
}
constexpr int kDppRowShr = 0x110, kDppRowRor = 0x120;   // + lanes
constexpr int kDppRowBcast15 = 0x142;   // lane 15 of each row to the next row
constexpr int kDppRowBcast31 = 0x143;   // lane 31 to rows 2 and 3

// The values of lanes l < 32 (WHICH 0) or l >= 32 (WHICH 1) for both l and
// l ^ 32, and the same for 16 within halves: op(WHICH 0, WHICH 1) combines
// every lane with its partner.
template <int WHICH, typename T>
__device__ __forceinline__ T half_of_pair32(T v) {
    return by_words(v, [](uint32_t x) { return (uint32_t)__builtin_amdgcn_permlane32_swap(x, x, false, false)[WHICH]; });
}
template <int WHICH, typename T>
__device__ __forceinline__ T half_of_pair16(T v) {
    return by_words(v, [](uint32_t x) { return (uint32_t)__builtin_amdgcn_permlane16_swap(x, x, false, false)[WHICH]; });
}

// v of all lanes combined by a commutative op, in the pairs of a butterfly over
// lane ^ 32, 16, 8, 4, 2, 1 (after step k the row repeats with period k, so
// that a rotation by k / 2 reads lane ^ k / 2).
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
    v = op(half_of_pair32<0>(v), half_of_pair32<1>(v));
    v = op(half_of_pair16<0>(v), half_of_pair16<1>(v));
    v = op(v, dpp_move<kDppRowRor + 8>(v));
    v = op(v, dpp_move<kDppRowRor + 4>(v));
    v = op(v, dpp_move<kDppRowRor + 2>(v));
    return op(v, dpp_move<kDppRowRor + 1>(v));
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    return wave_reduce(v, [](T a, T b) { return a + b; });
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
    return wave_reduce(v, [](T a, T b) { return a > b ? a : b; });
}
template <typename T>
__device__ __forceinline__ T wave_min(T v) {
    return wave_reduce(v, [](T a, T b) { return a < b ? a : b; });
}

// Inclusive scan of integers across the wave: within the rows, then the totals
// of the rows in front.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v) {
    static_assert(T(1) / T(2) == T(0), "whole numbers: the sums are grouped by rows");
    v += dpp_move<kDppRowShr + 1>(v);
    v += dpp_move<kDppRowShr + 2>(v);
    v += dpp_move<kDppRowShr + 4>(v);
    v += dpp_move<kDppRowShr + 8>(v);
    v += dpp_move<kDppRowBcast15, 0xA>(v);
    return v + dpp_move<kDppRowBcast31, 0xC>(v);
}

// Exclusive scan over a block of NT threads; returns the block total in *total.
// `scratch` must hold NT / 64 elements of T.
template <typename T, int NT>
__device__ __forceinline__ T block_exclusive_scan(T v, T *scratch, T *total) {
    static_assert(NT % kWave == 0, "block must be whole wavefronts");
    constexpr int NW = NT / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    T inc = wave_inclusive_scan(v);
    if (lane == kWave - 1) scratch[w] = inc;
    __syncthreads();
    T wave_off = 0, sum = 0;
#pragma unroll
    for (int k = 0; k < NW; k++) {
        const T s = scratch[k];
        if (k < w) wave_off += s;
        sum += s;
    }
    __syncthreads();
    *total = sum;
    return wave_off + inc - v;
}

template <typename T, int NT>
__device__ __forceinline__ T block_sum(T v, T *scratch) {
    constexpr int NW = NT / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    v = wave_sum(v);
    if (lane == 0) scratch[w] = v;
    __syncthreads();
    T sum = 0;
#pragma unroll
    for (int k = 0; k < NW; k++) sum += scratch[k];
    __syncthreads();
    return sum;
}

}  // namespace gsp

namespace gsp {

// DPP controls (gfx9 encoding) for row-local (16-lane) butterflies.
constexpr int kDppQuadXor1 = 0xB1;     // quad_perm [1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;     // quad_perm [2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;

// x + x[permuted lane]; every permutation used here reads a lane inside the
// row, so bound_ctrl (zero for out-of-range sources) never applies and lets
// the compiler fold the move into the add (v_add_f32_dpp).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Sum over the 16 lanes of each row; every lane of the row receives it.
__device__ __forceinline__ float row_sum16(float x) {
    x = dpp_add<kDppQuadXor1>(x);
    x = dpp_add<kDppQuadXor2>(x);
    x = dpp_add<kDppRowHalfMirror>(x);
    return dpp_add<kDppRowMirror>(x);
}

// (a, b) -> lanes 0-31: a[l] + a[l + 32]; lanes 32-63: b[l - 32] + b[l]
// (gfx950 v_permlane32_swap exchanges rows 2-3 of a with rows 0-1 of b).
__device__ __forceinline__ float pair_sum32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// (a, b) -> rows [a0 + a1, b0 + b1, a2 + a3, b2 + b3] (rows of 16 lanes;
// v_permlane16_swap exchanges the odd rows of a with the even rows of b).
__device__ __forceinline__ float pair_sum16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The first two levels of a reduce-scatter of nine values over the wave: a
// 32-lane and a 16-lane swap halve the data at each step, leaving each value
// as 16 partial sums (of the four lanes l, l + 16, l + 32, l + 48 of column
// l) in one 16-lane row:
//   a rows 0..3 = v0, v2, v1, v3;  b rows 0..3 = v4, v6, v5, v7;  c row 0 = v8.
__device__ __forceinline__ void wave_sum9_rows(const float v[9], float &a, float &b, float &c) {
    const float w0 = pair_sum32(v[0], v[1]);
    const float w1 = pair_sum32(v[2], v[3]);
    const float w2 = pair_sum32(v[4], v[5]);
    const float w3 = pair_sum32(v[6], v[7]);
    const float w4 = pair_sum32(v[8], v[8]);
    a = pair_sum16(w0, w1);
    b = pair_sum16(w2, w3);
    c = pair_sum16(w4, w4);
}

// The same for eight values: a rows 0..3 = v0, v2, v1, v3; b rows 0..3 =
// v4, v6, v5, v7.
__device__ __forceinline__ void wave_sum8_rows(const float v[8], float &a, float &b) {
    a = pair_sum16(pair_sum32(v[0], v[1]), pair_sum32(v[2], v[3]));
    b = pair_sum16(pair_sum32(v[4], v[5]), pair_sum32(v[6], v[7]));
}

// The same steps on doubles, then the sums over each row: six sums over the
// wave, each the value wave_sum gives (the same pairs in the same order), in
// half its operations.  a rows 0..3 = v0, v2, v1, v3; b rows 0, 1 = v4, rows 2,
// 3 = v5.
template <bool B32>
__device__ __forceinline__ double pair_sum_f64(double a, double b) {
    const uint32_t al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
    const auto lo = B32 ? __builtin_amdgcn_permlane32_swap(al, bl, false, false)
                        : __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto hi = B32 ? __builtin_amdgcn_permlane32_swap(ah, bh, false, false)
                        : __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

__device__ __forceinline__ void wave_sum6(const double v[6], double &a, double &b) {
    const double w = pair_sum_f64<true>(v[4], v[5]);
    a = pair_sum_f64<false>(pair_sum_f64<true>(v[0], v[1]), pair_sum_f64<true>(v[2], v[3]));
    b = pair_sum_f64<false>(w, w);
    a += dpp_move<kDppRowRor + 8>(a);
    b += dpp_move<kDppRowRor + 8>(b);
    a += dpp_move<kDppRowRor + 4>(a);
    b += dpp_move<kDppRowRor + 4>(b);
    a += dpp_move<kDppRowRor + 2>(a);
    b += dpp_move<kDppRowRor + 2>(b);
    a += dpp_move<kDppRowRor + 1>(a);
    b += dpp_move<kDppRowRor + 1>(b);
}

// Row of the 16-lane row partials that hold value k (register k >> 2 for
// k < 8, register 2 for k = 8).
__host__ __device__ constexpr int sum9_row(int k) {
    return k == 8 ? 0 : ((k & 3) == 1 ? 2 : ((k & 3) == 2 ? 1 : (k & 3)));
}

}  // namespace gsp
