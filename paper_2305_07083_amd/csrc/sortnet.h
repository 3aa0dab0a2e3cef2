// Compile-time sorting network over N keys held in registers.
//
// Batcher's merge exchange (Knuth, The Art of Computer Programming, vol. 3,
// 5.2.2, algorithm M): it sorts any N, not only powers of two, with every
// comparator putting the smaller key at the lower index, and takes a fifth to
// a quarter fewer comparators than a bitonic network (8, 12, 16, 24, 32 keys:
// 19, 41, 63, 127, 191 against 24, 54, 80, 168, 240).  The comparator list is a
// constant and its loop unrolls completely, so the key array never leaves
// registers.
#pragma once
#include <stdint.h>

namespace dfb {

// The comparators (a[c], b[c]), a[c] < b[c], of the network for N keys.
template <int N>
struct MergeExchange {
  int n = 0;
  int a[N * 10] = {}, b[N * 10] = {};
  constexpr MergeExchange() {
    int top = 1;
    while (2 * top < N) top *= 2;
    for (int p = N > 1 ? top : 0; p > 0; p /= 2) {
      int q = top, r = 0, d = p;
      for (;;) {
        for (int i = 0; i + d < N; ++i)
          if ((i & p) == r) {
            a[n] = i;
            b[n] = i + d;
            ++n;
          }
        if (q == p) break;
        d = q - p;
        q /= 2;
        r = p;
      }
    }
  }
};

template <typename K>
__host__ __device__ __forceinline__ void compare_exchange(K& a, K& b) {
  const bool lt = a < b;  // one compare, two selects per word
  const K lo = lt ? a : b;
  const K hi = lt ? b : a;
  a = lo;
  b = hi;
}

template <typename K>
struct CompareExchange {
  __host__ __device__ __forceinline__ void operator()(K& a, K& b) const { compare_exchange(a, b); }
};

// The network with a given comparator ce(a, b): min to a, max to b.
template <int N, typename K, typename CE>
__host__ __device__ __forceinline__ void sort_network(K (&k)[N], CE ce) {
  constexpr MergeExchange<N> net;
#pragma unroll
  for (int c = 0; c < net.n; ++c) ce(k[net.a[c]], k[net.b[c]]);
}

template <int N, typename K>
__host__ __device__ __forceinline__ void sort_network(K (&k)[N]) {
  sort_network<N>(k, CompareExchange<K>());
}

}  // namespace dfb
