// Sort of 16 R keys held by the 16 lanes of a DPP row, R per lane in
// registers: the lane of rank i ends with the sorted positions i R .. i R + R
// - 1.  Four rows of a wave sort four pixels at once, with no LDS traffic.
//
// Each lane sorts its R keys, then sequences of 1, 2, 4 and 8 lanes are merged
// in pairs: a stage that leaves two bitonic halves over the larger rank
// distance, half-cleaners over the smaller ones, then inside the lanes.  A
// half-cleaner splits a bitonic sequence of any even length into two bitonic
// halves, so inside a lane R may be 2^a or 3 2^a: a K just above a power of two
// does not pay for the next one.
//
// A comparator across lanes costs a DPP move a word and what makes one lane of
// the pair keep the minimum and the other the maximum:
//   32-bit keys: v_med3 with a limit below or above every key, by lane; two
//     instructions a key.  A rank is a lane number; the first stage of a merge
//     pairs positions with their mirror.
//   64-bit keys: there is no med3, but v_min_f64 takes a negated operand.  A
//     lane that has to keep the maximum holds its keys reversed (sign flipped),
//     and both take the minimum of their own key and the reversed partner:
//     three instructions a key.  Which lanes are reversed changes between two
//     distances, one exclusive-or a key.  The second sequence of a pair runs in
//     descending order, which is only another set of reversed lanes, so that
//     the first stage is a half-cleaner too; and ranks are numbered so that
//     every distance is one DPP move: rank bits 0, 1, 2 and 3 are lane
//     exchanges by xor 1, 2, 7 (row_half_mirror) and 8 (row_ror:8).  In lane
//     numbers distance 4 takes two moves a word.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sortnet.h"

namespace dfb {

// DPP controls of lane exchanges within a row of 16
constexpr int kLaneXor1 = 0xB1;    // quad_perm 1 0 3 2
constexpr int kLaneXor2 = 0x4E;    // quad_perm 2 3 0 1
constexpr int kLaneXor3 = 0x1B;    // quad_perm 3 2 1 0
constexpr int kLaneXor7 = 0x141;   // row_half_mirror
constexpr int kLaneXor8 = 0x128;   // row_ror:8
constexpr int kLaneXor15 = 0x140;  // row_mirror
constexpr int kLaneXor4 = -4;      // row_half_mirror, then quad_perm 3 2 1 0

template <int X>
__device__ __forceinline__ uint32_t lane_fetch(uint32_t v) {
  if constexpr (X == kLaneXor4) return lane_fetch<kLaneXor3>(lane_fetch<kLaneXor7>(v));
  else return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), X, 0xf, 0xf, true));
}

// Inclusive to exclusive scans and sums over a row of 16.
template <int N>
__device__ __forceinline__ float lane_shr_or(float v, float fill) {  // lane j takes lane j - N, or fill
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(fill), __float_as_int(v), 0x110 + N, 0xf, 0xf, false));
}
template <class RK>
__device__ __forceinline__ float row_product_before(float v) {  // product of the lanes of lower rank
  v = RK::by_rank(v);
  v *= lane_shr_or<1>(v, 1.f);
  v *= lane_shr_or<2>(v, 1.f);
  v *= lane_shr_or<4>(v, 1.f);
  v *= lane_shr_or<8>(v, 1.f);
  return RK::by_rank(lane_shr_or<1>(v, 1.f));
}
__device__ __forceinline__ float row_sum(float v) {  // in every lane
  v += __uint_as_float(lane_fetch<kLaneXor1>(__float_as_uint(v)));
  v += __uint_as_float(lane_fetch<kLaneXor2>(__float_as_uint(v)));
  v += __uint_as_float(lane_fetch<kLaneXor7>(__float_as_uint(v)));
  v += __uint_as_float(lane_fetch<kLaneXor15>(__float_as_uint(v)));
  return v;
}

// 64-bit keys that are the bit patterns of normal doubles of one sign.
struct RowKey64 {
  using K = uint64_t;
  static constexpr uint32_t kFlip = 0x80000000u;  // reversed: the sign bit
  // rank of lane j of a row, and the lane of a rank
  static __device__ __forceinline__ int rank(int j) { return (j & 4) ? j ^ 3 : j; }
  // v of the lane whose number is this lane's rank: the odd quads turned round
  static __device__ __forceinline__ float by_rank(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), kLaneXor3, 0xf, 0xa, false));
  }
  static __device__ __forceinline__ void ce(K& a, K& b) {
    const double x = __builtin_bit_cast(double, a), y = __builtin_bit_cast(double, b);
    double lo, hi;
    asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(x), "v"(y));
    asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(x), "v"(y));
    a = __builtin_bit_cast(K, lo);
    b = __builtin_bit_cast(K, hi);
  }
  static __device__ __forceinline__ K flip(K k, uint32_t m) { return k ^ (static_cast<uint64_t>(m) << 32); }
  template <int X>
  static __device__ __forceinline__ K fetch(K k) {
    return (static_cast<uint64_t>(lane_fetch<X>(static_cast<uint32_t>(k >> 32))) << 32) |
           lane_fetch<X>(static_cast<uint32_t>(k));
  }
  static __device__ __forceinline__ K min_reversed(K own, K other) {
    const double x = __builtin_bit_cast(double, own), y = __builtin_bit_cast(double, other);
    double r;
    asm("v_min_f64 %0, %1, -%2" : "=v"(r) : "v"(x), "v"(y));
    return __builtin_bit_cast(K, r);
  }
};

// 32-bit keys above INT32_MIN and below INT32_MAX.
struct RowKey32 {
  using K = int32_t;
  static __device__ __forceinline__ int rank(int j) { return j; }
  static __device__ __forceinline__ float by_rank(float v) { return v; }
  static __device__ __forceinline__ void ce(K& a, K& b) {
    const K lo = a < b ? a : b, hi = a < b ? b : a;
    a = lo;
    b = hi;
  }
  // the minimum (limit INT32_MIN) or the maximum (INT32_MAX) of the two
  template <int X>
  static __device__ __forceinline__ K keep(K own, K other, K limit) {
    const K x = static_cast<K>(lane_fetch<X>(static_cast<uint32_t>(other)));
    K r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(own), "v"(x), "v"(limit));
    return r;
  }
};

template <class RK>
struct RowCompare {
  __device__ __forceinline__ void operator()(typename RK::K& a, typename RK::K& b) const { RK::ce(a, b); }
};

// Sort of a bitonic sequence of N = 2^a or 3 2^a keys in a lane.
template <class RK, int N, int R>
__device__ __forceinline__ void lane_merge(typename RK::K (&k)[R]) {
  if constexpr (N % 2 == 0) {
#pragma unroll
    for (int b = 0; b < R; b += N)
#pragma unroll
      for (int i = 0; i < N / 2; ++i) RK::ce(k[b + i], k[b + i + N / 2]);
    lane_merge<RK, N / 2, R>(k);
  } else if constexpr (N == 3) {
#pragma unroll
    for (int b = 0; b < R; b += 3) {
      RK::ce(k[b], k[b + 2]);
      RK::ce(k[b], k[b + 1]);
      RK::ce(k[b + 1], k[b + 2]);
    }
  }
}

template <class RK, int R>
__device__ __forceinline__ void row_flip(typename RK::K (&k)[R], uint32_t m) {
#pragma unroll
  for (int r = 0; r < R; ++r) k[r] = RK::flip(k[r], m);
}
template <class RK, int R, int X>
__device__ __forceinline__ void row_clean(typename RK::K (&k)[R]) {
#pragma unroll
  for (int r = 0; r < R; ++r) k[r] = RK::min_reversed(k[r], RK::template fetch<X>(k[r]));
}

// Keys of odd ranks come reversed (the sign bit of RowKey64::kFlip set).
template <class RK, int R>
__device__ __forceinline__ void row_sort(uint64_t (&k)[R], int lane) {
  const int rank = RK::rank(lane & 15);
  uint32_t m[4];  // lanes whose keys are reversed at rank distance 2^b, or whose sequence of 2^b lanes descends
#pragma unroll
  for (int b = 0; b < 4; ++b) m[b] = (rank >> b) & 1 ? RK::kFlip : 0u;
  sort_network<R>(k, RowCompare<RK>());
  row_flip<RK>(k, m[1]);
  row_clean<RK, R, kLaneXor1>(k);
  row_flip<RK>(k, m[0]);
  lane_merge<RK, R>(k);
  row_flip<RK>(k, m[2]);
  row_clean<RK, R, kLaneXor2>(k);
  row_flip<RK>(k, m[1] ^ m[0]);
  row_clean<RK, R, kLaneXor1>(k);
  row_flip<RK>(k, m[0]);
  lane_merge<RK, R>(k);
  row_flip<RK>(k, m[3]);
  row_clean<RK, R, kLaneXor7>(k);
  row_flip<RK>(k, m[2] ^ m[1]);
  row_clean<RK, R, kLaneXor2>(k);
  row_flip<RK>(k, m[1] ^ m[0]);
  row_clean<RK, R, kLaneXor1>(k);
  row_flip<RK>(k, m[0]);
  lane_merge<RK, R>(k);
  row_clean<RK, R, kLaneXor8>(k);
  row_flip<RK>(k, m[3] ^ m[2]);
  row_clean<RK, R, kLaneXor7>(k);
  row_flip<RK>(k, m[2] ^ m[1]);
  row_clean<RK, R, kLaneXor2>(k);
  row_flip<RK>(k, m[1] ^ m[0]);
  row_clean<RK, R, kLaneXor1>(k);
  row_flip<RK>(k, m[0]);
  lane_merge<RK, R>(k);
}

template <int R, int X>
__device__ __forceinline__ void row_keep(int32_t (&k)[R], int32_t limit) {
#pragma unroll
  for (int r = 0; r < R; ++r) k[r] = RowKey32::keep<X>(k[r], k[r], limit);
}
template <int R, int X>
__device__ __forceinline__ void row_keep_mirror(int32_t (&k)[R], int32_t limit) {
#pragma unroll
  for (int r = 0; r < R / 2; ++r) {
    const int32_t a = k[r], b = k[R - 1 - r];
    k[r] = RowKey32::keep<X>(a, b, limit);
    k[R - 1 - r] = RowKey32::keep<X>(b, a, limit);
  }
}
template <class RK, int R>
__device__ __forceinline__ void row_sort(int32_t (&k)[R], int lane) {
  static_assert(R % 2 == 0, "the mirrored stage pairs a lane's keys");
  int32_t lim[4];  // of the lanes that keep the maximum at distance 2^b, and of the others
#pragma unroll
  for (int b = 0; b < 4; ++b) lim[b] = (lane >> b) & 1 ? INT32_MAX : INT32_MIN;
  sort_network<R>(k, RowCompare<RK>());
  row_keep_mirror<R, kLaneXor1>(k, lim[0]);
  lane_merge<RK, R>(k);
  row_keep_mirror<R, kLaneXor3>(k, lim[1]);
  row_keep<R, kLaneXor1>(k, lim[0]);
  lane_merge<RK, R>(k);
  row_keep_mirror<R, kLaneXor7>(k, lim[2]);
  row_keep<R, kLaneXor2>(k, lim[1]);
  row_keep<R, kLaneXor1>(k, lim[0]);
  lane_merge<RK, R>(k);
  row_keep_mirror<R, kLaneXor15>(k, lim[3]);
  row_keep<R, kLaneXor4>(k, lim[2]);
  row_keep<R, kLaneXor2>(k, lim[1]);
  row_keep<R, kLaneXor1>(k, lim[0]);
  lane_merge<RK, R>(k);
}

}  // namespace dfb
