// gfx950 kernels of the per-tile sort-last compositor.
//
// One to three persistent launches per frame (by the layer counts of its
// tiles).  Each workgroup (64 * waves_per_tile lanes) repeatedly takes a work unit -- a work_w x work_h rectangle of one DFB tile
// -- from a device queue ordered longest tile first, and for every pixel of it
//   1. builds the key (ordered depth bits << 32 | layer index) of each of the
//      tile's K layers from coalesced SoA depth loads, staging alpha in LDS,
//   2. sorts the keys (a lane's registers for K <= 32, the registers of 16
//      lanes for K <= 512, an LDS bitonic sort shared by the workgroup above),
//   3. walks the sorted keys front to back computing the transmittance T in
//      front of each layer ("over", Sec. 4.2 of the paper) and writes it back
//      into the layer's LDS slot,
//   4. sums T_l * colour_l in layer order with coalesced colour loads and puts
//      the background behind (the generation-0 tile),
//   5. optionally stores the finished f32 pixel, folds it into the running
//      mean and M2 (Welford) and tonemaps the displayed value to RGBA8.
// Per-tile variance: a wave/LDS reduction of M2 over the unit; units of one
// tile combine their partial sums in a fixed order (deterministic).
// Every fragment byte is read from HBM exactly once.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "dfb_internal.h"
#include "rowsort.h"
#include "sortnet.h"

namespace dfb {
namespace {

// Fragment planes are read exactly once per frame: streaming (non-temporal)
// loads keep them from displacing the outputs in L2.
#ifndef DFB_NT_LOADS
#define DFB_NT_LOADS 1
#endif
// Minimum waves per SIMD requested from the register allocator, per
// register-sort capacity (0 = no request).
#ifndef DFB_WAVES_K8
#define DFB_WAVES_K8 0
#endif
#ifndef DFB_WAVES_K16
#define DFB_WAVES_K16 0
#endif
#ifndef DFB_WAVES_K32
#define DFB_WAVES_K32 0
#endif
// Largest register-sort bucket that loads all five planes up front (larger
// buckets load depth and alpha first and the colours after the walk);
// 0 = chosen per kernel capacity (upfront_max).
#ifndef DFB_UPFRONT_MAX
#define DFB_UPFRONT_MAX 0
#endif
// Streaming (non-temporal) loads in the LDS sort too (1), or ordinary loads
// (0, the default): those leave a line in L2 for the pixel group that reads
// its other half (a group of 16 or fewer fp32 pixels covers half a 128-byte
// line or less); 36.5 against 38.6 ms on the 8192^2 heavy-tailed frame when
// this sort took all its tiles of more than 32 layers.
#ifndef DFB_BIGK_NT
#define DFB_BIGK_NT 0
#endif
// Layers whose plane loads the list and averaging operations keep in flight
// per lane.
#ifndef DFB_OP_CHUNK
#define DFB_OP_CHUNK 4
#endif

// Plane loads: `base` is uniform across the wave (a layer's block start) and
// `i` a 32-bit element offset inside the block, so each load is one
// instruction with a scalar base address.
template <typename FT>
__device__ __forceinline__ float ldf(const FT* __restrict__ base, uint32_t i);
template <>
__device__ __forceinline__ float ldf<float>(const float* __restrict__ base, uint32_t i) {
#if DFB_NT_LOADS
  return __builtin_nontemporal_load(base + i);
#else
  return base[i];
#endif
}
template <>
__device__ __forceinline__ float ldf<_Float16>(const _Float16* __restrict__ base, uint32_t i) {
#if DFB_NT_LOADS
  return static_cast<float>(__builtin_nontemporal_load(base + i));
#else
  return static_cast<float>(base[i]);
#endif
}

// Workgroup barrier for LDS traffic only.  Threads of a workgroup share
// nothing through global memory inside these kernels, so a barrier need not
// wait for the wave's global stores to complete (which __syncthreads does:
// that wait costs a memory round trip at every unit boundary).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Order-preserving map of a depth to 32 bits: NaN above everything, -0 == +0.
__device__ __forceinline__ uint32_t depth_bits(float d) {
  uint32_t b = __float_as_uint(d);
  if (d != d) return 0xFFFFFFFFu;
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Order-preserving map of a binary16 depth to 16 bits, same rules.
__device__ __forceinline__ uint32_t half_depth_bits(uint16_t h) {
  if ((h & 0x7C00u) == 0x7C00u && (h & 0x03FFu)) return 0xFFFFu;
  if (h == 0x8000u) h = 0;
  return (h & 0x8000u) ? (~static_cast<uint32_t>(h) & 0xFFFFu) : (static_cast<uint32_t>(h) | 0x8000u);
}

// Keys of fp32 depths.  The sort order (ordered depth bits, then layer
// index) is that of the 44-bit integer x = depth_bits << 12 | l (l < 4096).  Held as
// the double 2^52 + x (bit pattern 0x433 << 52 | x), every key is a normal
// double whose value orders like x, so a comparator is one v_min_f64 and one
// v_max_f64 instead of two 64-bit integer compares and four selects.  The
// layer index is the low 12 bits of the pattern.
constexpr uint64_t kKeyBias = 0x4330000000000000ull;
constexpr uint64_t kKeyPad = kKeyBias | 0x00000FFFFFFFFFFFull;  // not below any real key
__device__ __forceinline__ uint64_t big_key(uint32_t dbits, int l) {
  return kKeyBias | (static_cast<uint64_t>(dbits) << 12) | static_cast<uint32_t>(l);
}
__device__ __forceinline__ int key_layer(uint64_t k) { return static_cast<int>(k & 0xFFFu); }
struct KeyMinMax {
  __device__ __forceinline__ void operator()(uint64_t& a, uint64_t& b) const {
    const double x = __builtin_bit_cast(double, a), y = __builtin_bit_cast(double, b);
    double lo, hi;
    asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(x), "v"(y));
    asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(x), "v"(y));
    a = __builtin_bit_cast(uint64_t, lo);
    b = __builtin_bit_cast(uint64_t, hi);
  }
};

// Sort keys of the register path: (ordered depth bits, layer index), as one
// number so that one comparison orders by depth and breaks ties by index (the
// layers of a tile are in source-id order).  fp32 depths take the 64-bit
// double-encoded key above; fp16 depths and an index below 65536 fit 32 bits
// (v_min_u32 / v_max_u32), which also halves the registers.
template <typename FT>
struct SortKey;
template <>
struct SortKey<float> {
  using K = uint64_t;
  using CE = KeyMinMax;
  static constexpr K kPad = kKeyPad;
  __device__ static __forceinline__ K make(const float* __restrict__ b, uint32_t i, int l) {
    return big_key(depth_bits(ldf<float>(b, i)), l);
  }
  __device__ static __forceinline__ int index(K k) { return key_layer(k); }
};
template <>
struct SortKey<_Float16> {
  using K = uint32_t;
  using CE = CompareExchange<uint32_t>;
  static constexpr K kPad = ~0u;
  __device__ static __forceinline__ K make(const _Float16* __restrict__ b, uint32_t i, int l) {
#if DFB_NT_LOADS
    const _Float16 d = __builtin_nontemporal_load(b + i);
#else
    const _Float16 d = b[i];
#endif
    return (half_depth_bits(__builtin_bit_cast(uint16_t, d)) << 16) | static_cast<uint32_t>(l);
  }
  __device__ static __forceinline__ int index(K k) { return static_cast<int>(k & 0xFFFFu); }
};

__device__ __forceinline__ uint32_t quantise(float x, bool gamma, float inv_gamma) {
  float y = x > 0.f ? x : 0.f;  // NaN compares false -> 0
  y = y < 1.f ? y : 1.f;
  if (gamma) y = powf(y, inv_gamma);
  return static_cast<uint32_t>(floorf(fmaf(255.f, y, 0.5f)));
}

__device__ __forceinline__ uint32_t pack_rgba8(float4 v, uint32_t mode, float inv_gamma) {
  const bool g = (mode & kModeGamma) != 0;
  return quantise(v.x, g, inv_gamma) | (quantise(v.y, g, inv_gamma) << 8) |
         (quantise(v.z, g, inv_gamma) << 16) | (quantise(v.w, false, 1.f) << 24);
}

// Pixel -> finished / accumulated / displayed outputs.  Returns the pixel's
// M2 sum over RGB (0 when not accumulating or outside the image).
__device__ __forceinline__ float store_pixel(float4 x, size_t px, size_t m2_base, int P,
                                             bool inside, uint32_t mode, int n_acc, float inv_n,
                                             float inv_gamma, float* finished, float* accum,
                                             float* m2, void* final_out) {
  if (mode & kModeKeepFinished) reinterpret_cast<float4*>(finished)[px] = x;
  float4 disp = x;
  float vs = 0.f;
  if (mode & kModeAccumulate) {
    float* q = m2 + m2_base;
    float4 mu;
    float q0, q1, q2;
    if (n_acc == 1) {
      mu = x;
      q0 = q1 = q2 = 0.f;
    } else {
      mu = reinterpret_cast<const float4*>(accum)[px];
      q0 = q[0];
      q1 = q[P];
      q2 = q[2 * P];
      const float d0 = x.x - mu.x, d1 = x.y - mu.y, d2 = x.z - mu.z, d3 = x.w - mu.w;
      mu.x = fmaf(d0, inv_n, mu.x);
      mu.y = fmaf(d1, inv_n, mu.y);
      mu.z = fmaf(d2, inv_n, mu.z);
      mu.w = fmaf(d3, inv_n, mu.w);
      q0 = fmaf(d0, x.x - mu.x, q0);
      q1 = fmaf(d1, x.y - mu.y, q1);
      q2 = fmaf(d2, x.z - mu.z, q2);
    }
    reinterpret_cast<float4*>(accum)[px] = mu;
    q[0] = q0;
    q[P] = q1;
    q[2 * P] = q2;
    if (inside) vs = q0 + q1 + q2;
    disp = mu;
  }
  if (mode & kModeFmtRGBA8) {
    static_cast<uint32_t*>(final_out)[px] = pack_rgba8(disp, mode, inv_gamma);
  } else if (mode & kModeFmtF32) {
    static_cast<float4*>(final_out)[px] = disp;
  }
  return vs;
}

struct Unit {
  int t, sx0, sy0, x0, y0;  // tile, unit origin inside the tile, tile origin in the image
};

__device__ __forceinline__ int unit_pixel(const FrameArgs& a, const Unit& u, int q, bool& inside) {
  const int qy = a.work_shift >= 0 ? (q >> a.work_shift) : q / a.work_w;
  const int qx = q - qy * a.work_w;
  const int ty = u.sy0 + qy, tx = u.sx0 + qx;
  inside = (u.x0 + tx < a.width) && (u.y0 + ty < a.height);
  return ty * a.tile_w + tx;
}

__device__ __forceinline__ float finish_px(const FrameArgs& a, const Unit& u, int p, bool inside,
                                           float4 x) {
  const size_t px = static_cast<size_t>(u.t) * a.P + p;
  const size_t mb = static_cast<size_t>(u.t) * 3 * a.P + p;
  return store_pixel(x, px, mb, a.P, inside, a.mode, a.n_acc, a.inv_n, a.inv_gamma, a.finished,
                     a.accum, a.m2, a.final_out);
}

// ---------------------------------------------------------------- K <= 32
// One lane per pixel.  All five planes of the pixel's K fragments are loaded
// up front (one memory round trip per pixel, 5K loads in flight); colours
// stay in registers indexed by layer, so only the sorted walk needs dynamic
// indexing: wl points at this lane's column of a [KMAX][NT] LDS array, the
// lane writes alpha of layer l to wl[l*NT] and the walk overwrites it with
// the transmittance in front of layer l.  No lane reads another lane's
// column, so no barrier is needed.
template <typename FT, int KMAX>
__device__ __forceinline__ float4 composite_px_upfront(float& Tout, const FrameArgs& a,
                                                       const int64_t* __restrict__ loff, int K,
                                                       int off, int p, float* __restrict__ wl,
                                                       int NT) {
  const uint32_t P = static_cast<uint32_t>(a.P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  const uint32_t up = static_cast<uint32_t>(p);
  using SK = SortKey<FT>;
  typename SK::K key[KMAX];
  float alp[KMAX], cr[KMAX], cg[KMAX], cb[KMAX];
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    if (l < K) {
      const FT* __restrict__ b = frag + loff[l];
      key[l] = SK::make(b, 4 * P + up, l);
      alp[l] = ldf<FT>(b, 3 * P + up);
      cr[l] = ldf<FT>(b, up);
      cg[l] = ldf<FT>(b, P + up);
      cb[l] = ldf<FT>(b, 2 * P + up);
    } else {
      key[l] = SK::kPad;
    }
  }
#pragma unroll
  for (int l = 0; l < KMAX; ++l)
    if (l < K) wl[l * NT] = alp[l];
  sort_network<KMAX>(key, typename SK::CE());
  float T = 1.f, A = 0.f;
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    if (i < K) {
      const int l = SK::index(key[i]);
      const float al = wl[l * NT];
      wl[l * NT] = T;
      A = fmaf(T, al, A);
      T = T * (1.f - al);
      if (a.mode & kModeKeepOrder)
        a.order[static_cast<size_t>(off + i) * P + p] = static_cast<uint16_t>(l);
    }
  }
  float R = 0.f, G = 0.f, B = 0.f;
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    if (l < K) {
      const float w = wl[l * NT];
      R = fmaf(w, cr[l], R);
      G = fmaf(w, cg[l], G);
      B = fmaf(w, cb[l], B);
    }
  }
  Tout = T;
  return make_float4(R, G, B, A);
}

// Larger K: 5K values per lane no longer fit the register file next to the
// keys, so depth and alpha are loaded first and the colours only after the
// walk (two memory round trips per pixel, half the registers).
template <typename FT, int KMAX>
__device__ __forceinline__ float4 composite_px_two_phase(float& Tout, const FrameArgs& a,
                                                         const int64_t* __restrict__ loff, int K,
                                                         int off, int p, float* __restrict__ wl,
                                                         int NT) {
  const uint32_t P = static_cast<uint32_t>(a.P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  const uint32_t up = static_cast<uint32_t>(p);
  using SK = SortKey<FT>;
  typename SK::K key[KMAX];
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    if (l < K) {
      const FT* __restrict__ b = frag + loff[l];
      key[l] = SK::make(b, 4 * P + up, l);
      wl[l * NT] = ldf<FT>(b, 3 * P + up);
    } else {
      key[l] = SK::kPad;
    }
  }
  sort_network<KMAX>(key, typename SK::CE());
  float T = 1.f, A = 0.f;
#pragma unroll
  for (int i = 0; i < KMAX; ++i) {
    if (i < K) {
      const int l = SK::index(key[i]);
      const float al = wl[l * NT];
      wl[l * NT] = T;
      A = fmaf(T, al, A);
      T = T * (1.f - al);
      if (a.mode & kModeKeepOrder)
        a.order[static_cast<size_t>(off + i) * P + p] = static_cast<uint16_t>(l);
    }
  }
  float R = 0.f, G = 0.f, B = 0.f;
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    if (l < K) {
      const FT* __restrict__ b = frag + loff[l];
      const float w = wl[l * NT];
      R = fmaf(w, ldf<FT>(b, up), R);
      G = fmaf(w, ldf<FT>(b, P + up), G);
      B = fmaf(w, ldf<FT>(b, 2 * P + up), B);
    }
  }
  Tout = T;
  return make_float4(R, G, B, A);
}

// Up-front loads for buckets up to upfront_max(KCAP): one memory round trip
// per pixel instead of two, at the cost of registers.  The fp32 16-layer
// kernel stays at 3 waves per SIMD with all its buckets up front (2048^2
// bricks: 139 against 144 us); the fp16 one would drop from 4 to 3, so its
// 12/16 buckets load in two phases.  The fp32 32-layer kernel stays at 2
// waves with the 24 bucket up front (4096x1024: 225 against 232 us); its 32
// bucket loads in two phases.  The fp16 32-layer kernel loads up to 12
// layers up front: 168 VGPRs, 3 waves per SIMD instead of 2 with the 24
// bucket up front (211 VGPRs): the 4096x1024 fp16 frame takes 164 instead of
// 186 us.
#ifndef DFB_UPFRONT_F16_K32
#define DFB_UPFRONT_F16_K32 12   // largest up-front bucket of the fp16 32-layer kernel
#endif
template <typename FT>
constexpr int upfront_max(int kcap) {
  return DFB_UPFRONT_MAX > 0 ? DFB_UPFRONT_MAX
                             : (kcap <= 16 ? (sizeof(FT) == 4 ? 16 : 8) : (sizeof(FT) == 4 ? 24 : DFB_UPFRONT_F16_K32));
}

template <typename FT, int KMAX, int KCAP>
__device__ __forceinline__ float4 composite_px(float& T, const FrameArgs& a, const int64_t* __restrict__ loff,
                                               int K, int off, int p, float* __restrict__ wl,
                                               int NT) {
  if constexpr (KMAX <= upfront_max<FT>(KCAP)) return composite_px_upfront<FT, KMAX>(T, a, loff, K, off, p, wl, NT);
  else return composite_px_two_phase<FT, KMAX>(T, a, loff, K, off, p, wl, NT);
}

// The background (the generation-0 tile) behind whatever transmittance T is
// left: a constant colour, or a per-pixel image when one is configured.
__device__ __forceinline__ float4 with_background(const FrameArgs& a, int t, int p, float4 x, float T) {
  float4 bg;
  if (a.bg_image) {
    bg = reinterpret_cast<const float4*>(a.bg_image)[static_cast<size_t>(t) * a.P + p];
  } else {
    bg = make_float4(a.bg[0], a.bg[1], a.bg[2], a.bg[3]);
  }
  return make_float4(fmaf(T, bg.x, x.x), fmaf(T, bg.y, x.y), fmaf(T, bg.z, x.z), fmaf(T, bg.w, x.w));
}

template <typename FT, int KMAX, int KCAP>
__device__ float unit_reg(const FrameArgs& a, const Unit& u, const int64_t* __restrict__ loff, int K, int off,
                          float* lds) {
  static_assert(KMAX <= KCAP, "bucket within the kernel's capacity");
  const int NT = blockDim.x, tid = threadIdx.x;
  float vs = 0.f;
  for (int q = tid; q < a.work_px; q += NT) {
    bool inside;
    const int p = unit_pixel(a, u, q, inside);
    float T;
    const float4 x = composite_px<FT, KMAX, KCAP>(T, a, loff, K, off, p, lds + tid, NT);
    vs += finish_px(a, u, p, inside, with_background(a, u.t, p, x, T));
  }
  return vs;
}

__device__ float unit_background(const FrameArgs& a, const Unit& u) {
  const int NT = blockDim.x;
  float vs = 0.f;
  for (int q = threadIdx.x; q < a.work_px; q += NT) {
    bool inside;
    const int p = unit_pixel(a, u, q, inside);
    vs += finish_px(a, u, p, inside, with_background(a, u.t, p, make_float4(0.f, 0.f, 0.f, 0.f), 1.f));
  }
  return vs;
}

// Rank-order list (the paper's alternative when a per-rank order is correct):
// the tile's layers, ordered by generation (their source_id) back to front,
// are blended front to back from the highest generation down -- no depth is
// read and nothing is sorted.
template <typename FT>
__device__ float unit_list(const FrameArgs& a, const Unit& u, const int64_t* __restrict__ loff, int K,
                           int off) {
  const int NT = blockDim.x;
  const uint32_t P = static_cast<uint32_t>(a.P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  float vs = 0.f;
  for (int q = threadIdx.x; q < a.work_px; q += NT) {
    bool inside;
    const int p = unit_pixel(a, u, q, inside);
    const uint32_t up = static_cast<uint32_t>(p);
    float R = 0.f, G = 0.f, B = 0.f, A = 0.f, T = 1.f;
    int i = 0;
    for (; i + 4 <= K; i += 4) {  // 4 layers' loads in flight
      float cr[4], cg[4], cb[4], al[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const FT* __restrict__ b = frag + loff[K - 1 - (i + j)];
        cr[j] = ldf<FT>(b, up);
        cg[j] = ldf<FT>(b, P + up);
        cb[j] = ldf<FT>(b, 2 * P + up);
        al[j] = ldf<FT>(b, 3 * P + up);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        R = fmaf(T, cr[j], R);
        G = fmaf(T, cg[j], G);
        B = fmaf(T, cb[j], B);
        A = fmaf(T, al[j], A);
        T = T * (1.f - al[j]);
        if (a.mode & kModeKeepOrder)
          a.order[static_cast<size_t>(off + i + j) * P + p] = static_cast<uint16_t>(K - 1 - (i + j));
      }
    }
    for (; i < K; ++i) {
      const FT* __restrict__ b = frag + loff[K - 1 - i];
      const float al = ldf<FT>(b, 3 * P + up);
      R = fmaf(T, ldf<FT>(b, up), R);
      G = fmaf(T, ldf<FT>(b, P + up), G);
      B = fmaf(T, ldf<FT>(b, 2 * P + up), B);
      A = fmaf(T, al, A);
      T = T * (1.f - al);
      if (a.mode & kModeKeepOrder)
        a.order[static_cast<size_t>(off + i) * P + p] = static_cast<uint16_t>(K - 1 - i);
    }
    vs += finish_px(a, u, p, inside, with_background(a, u.t, p, make_float4(R, G, B, A), T));
  }
  return vs;
}

// 16-byte plane loads: V consecutive elements of one plane (4 fp32 or 8
// fp16 pixels), converted to float.  The element offset is a multiple of V
// and the block start is 16-byte aligned (checked on the host).
template <typename FT>
struct VecWidth;
template <>
struct VecWidth<float> {
  static constexpr int V = 4;
};
template <>
struct VecWidth<_Float16> {
  static constexpr int V = 8;
};

template <typename FT>
__device__ __forceinline__ void ldv(const FT* __restrict__ base, uint32_t i, float* out);
template <>
__device__ __forceinline__ void ldv<float>(const float* __restrict__ base, uint32_t i, float* out) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const f4 v = __builtin_nontemporal_load(reinterpret_cast<const f4*>(base + i));
  out[0] = v.x;
  out[1] = v.y;
  out[2] = v.z;
  out[3] = v.w;
}
template <>
__device__ __forceinline__ void ldv<_Float16>(const _Float16* __restrict__ base, uint32_t i, float* out) {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  const h8 v = __builtin_nontemporal_load(reinterpret_cast<const h8*>(base + i));
#pragma unroll
  for (int k = 0; k < 8; ++k) out[k] = static_cast<float>(v[k]);
}

// Block offsets of a tile's layers [base, base + 64) held one per lane, so a
// layer's offset is a register read (no dependent scalar load in the loop).
__device__ __forceinline__ int64_t lane_offsets(const int64_t* __restrict__ loff, int base, int K) {
  const int l = base + static_cast<int>(__lane_id());
  return (l >= 0 && l < K) ? loff[l] : 0;
}
__device__ __forceinline__ int64_t offset_of(int64_t held, int k) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(held), k);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(static_cast<uint64_t>(held) >> 32), k);
  return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

// V pixels of one unit row per lane; the finished pixels go through the same
// per-pixel epilogue as the scalar path.
template <int V, bool BG>
__device__ __forceinline__ float finish_row(const FrameArgs& a, const Unit& u, int q0, int p0, const float* R,
                                            const float* G, const float* B, const float* A, const float* T) {
  float vs = 0.f;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    bool inside;
    unit_pixel(a, u, q0 + v, inside);
    float4 x = make_float4(R[v], G[v], B[v], A[v]);
    if constexpr (BG) x = with_background(a, u.t, p0 + v, x, T[v]);
    vs += finish_px(a, u, p0 + v, inside, x);
  }
  return vs;
}

// The list operation with 16-byte loads: C layers' four planes in flight per
// lane, blended front to back from the highest generation.
template <typename FT>
__device__ float unit_list_vec(const FrameArgs& a, const Unit& u, const int64_t* __restrict__ loff, int K,
                               int off) {
  constexpr int V = VecWidth<FT>::V;
  constexpr int C = DFB_OP_CHUNK;
  const int NT = blockDim.x;
  const uint32_t P = static_cast<uint32_t>(a.P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  float vs = 0.f;
  // whole waves run the loop (the held offsets need every lane); lanes past
  // the unit's end load a valid row again and store nothing
  const int lane = static_cast<int>(threadIdx.x & 63);
  for (int base = static_cast<int>(threadIdx.x >> 6) * 64 * V; base < a.work_px; base += NT * V) {
    const bool act = base + lane * V < a.work_px;
    const int q0 = act ? base + lane * V : base;
    bool in0;
    const int p0 = unit_pixel(a, u, q0, in0);
    const uint32_t up = static_cast<uint32_t>(p0);
    float R[V], G[V], B[V], A[V], T[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      R[v] = G[v] = B[v] = A[v] = 0.f;
      T[v] = 1.f;
    }
    int i = 0;
    int64_t held = 0;
    for (; i + C <= K; i += C) {
      if ((i & 63) == 0) held = lane_offsets(loff, K - 64 - i, K);  // layers K-64-i .. K-1-i
      float x[C][4][V];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const FT* __restrict__ b = frag + offset_of(held, 63 - ((i + j) & 63));
#pragma unroll
        for (int c = 0; c < 4; ++c) ldv<FT>(b, c * P + up, x[j][c]);
      }
#pragma unroll
      for (int j = 0; j < C; ++j) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          R[v] = fmaf(T[v], x[j][0][v], R[v]);
          G[v] = fmaf(T[v], x[j][1][v], G[v]);
          B[v] = fmaf(T[v], x[j][2][v], B[v]);
          A[v] = fmaf(T[v], x[j][3][v], A[v]);
          T[v] = T[v] * (1.f - x[j][3][v]);
        }
        if ((a.mode & kModeKeepOrder) && act) {
#pragma unroll
          for (int v = 0; v < V; ++v)
            a.order[static_cast<size_t>(off + i + j) * P + p0 + v] = static_cast<uint16_t>(K - 1 - (i + j));
        }
      }
    }
    for (; i < K; ++i) {
      if ((i & 63) == 0) held = lane_offsets(loff, K - 64 - i, K);
      float x[4][V];
      const FT* __restrict__ b = frag + offset_of(held, 63 - (i & 63));
#pragma unroll
      for (int c = 0; c < 4; ++c) ldv<FT>(b, c * P + up, x[c]);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        R[v] = fmaf(T[v], x[0][v], R[v]);
        G[v] = fmaf(T[v], x[1][v], G[v]);
        B[v] = fmaf(T[v], x[2][v], B[v]);
        A[v] = fmaf(T[v], x[3][v], A[v]);
        T[v] = T[v] * (1.f - x[3][v]);
      }
      if ((a.mode & kModeKeepOrder) && act) {
#pragma unroll
        for (int v = 0; v < V; ++v)
          a.order[static_cast<size_t>(off + i) * P + p0 + v] = static_cast<uint16_t>(K - 1 - i);
      }
    }
    if (act) vs += finish_row<V, true>(a, u, q0, p0, R, G, B, A, T);
  }
  return vs;
}

// The averaging operation with 16-byte loads (layers summed in layer order;
// K > 0: a tile without renders is the background, handled by the caller).
template <typename FT>
__device__ float unit_average_vec(const FrameArgs& a, const Unit& u, const int64_t* __restrict__ loff, int K) {
  constexpr int V = VecWidth<FT>::V;
  constexpr int C = DFB_OP_CHUNK;
  const int NT = blockDim.x;
  const uint32_t P = static_cast<uint32_t>(a.P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  const float inv = K > 0 ? 1.f / static_cast<float>(K) : 0.f;
  float vs = 0.f;
  // whole waves run the loop (the held offsets need every lane); lanes past
  // the unit's end load a valid row again and store nothing
  const int lane = static_cast<int>(threadIdx.x & 63);
  for (int base = static_cast<int>(threadIdx.x >> 6) * 64 * V; base < a.work_px; base += NT * V) {
    const bool act = base + lane * V < a.work_px;
    const int q0 = act ? base + lane * V : base;
    bool in0;
    const int p0 = unit_pixel(a, u, q0, in0);
    const uint32_t up = static_cast<uint32_t>(p0);
    float S[4][V];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < V; ++v) S[c][v] = 0.f;
    int l = 0;
    int64_t held = 0;
    for (; l + C <= K; l += C) {
      if ((l & 63) == 0) held = lane_offsets(loff, l, K);
      float x[C][4][V];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const FT* __restrict__ b = frag + offset_of(held, (l + j) & 63);
#pragma unroll
        for (int c = 0; c < 4; ++c) ldv<FT>(b, c * P + up, x[j][c]);
      }
#pragma unroll
      for (int j = 0; j < C; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int v = 0; v < V; ++v) S[c][v] += x[j][c][v];
    }
    for (; l < K; ++l) {
      if ((l & 63) == 0) held = lane_offsets(loff, l, K);
      float x[4][V];
      const FT* __restrict__ b = frag + offset_of(held, l & 63);
#pragma unroll
      for (int c = 0; c < 4; ++c) ldv<FT>(b, c * P + up, x[c]);
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int v = 0; v < V; ++v) S[c][v] += x[c][v];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < V; ++v) S[c][v] *= inv;
    if (act) vs += finish_row<V, false>(a, u, q0, p0, S[0], S[1], S[2], S[3], nullptr);
  }
  return vs;
}

// Averaging tile operation (redundant sampling, the paper's dynamic load
// balancing): the finished pixel is the mean of the K tiles' RGBA; a tile
// with no layers shows the background.
template <typename FT>
__device__ float unit_average(const FrameArgs& a, const Unit& u, const int64_t* __restrict__ loff, int K) {
  const int NT = blockDim.x;
  const uint32_t P = static_cast<uint32_t>(a.P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  const float inv = K > 0 ? 1.f / static_cast<float>(K) : 0.f;
  float vs = 0.f;
  for (int q = threadIdx.x; q < a.work_px; q += NT) {
    bool inside;
    const int p = unit_pixel(a, u, q, inside);
    const uint32_t up = static_cast<uint32_t>(p);
    float R = 0.f, G = 0.f, B = 0.f, A = 0.f;
    int l = 0;
    for (; l + 4 <= K; l += 4) {
      float v[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const FT* __restrict__ b = frag + loff[l + j];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[j][c] = ldf<FT>(b, c * P + up);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        R += v[j][0];
        G += v[j][1];
        B += v[j][2];
        A += v[j][3];
      }
    }
    for (; l < K; ++l) {
      const FT* __restrict__ b = frag + loff[l];
      R += ldf<FT>(b, up);
      G += ldf<FT>(b, P + up);
      B += ldf<FT>(b, 2 * P + up);
      A += ldf<FT>(b, 3 * P + up);
    }
    const float4 x = K > 0 ? make_float4(R * inv, G * inv, B * inv, A * inv)
                           : with_background(a, u.t, p, make_float4(0.f, 0.f, 0.f, 0.f), 1.f);
    vs += finish_px(a, u, p, inside, x);
  }
  return vs;
}

// --------------------------------------------------------------- K > 512
// (and K > 32 where the planes are not 4-pixel aligned: the row sort below
// takes the others.)  The workgroup handles G pixels at a time.  LDS holds one row per pixel:
// Kp keys (u64) and, in a second array of the same shape, Kp floats (alpha,
// later the transmittance T); and the unit's layer offsets.  Position i of a
// row is stored at i + i/16 (one pad slot per 16) and rows are
// RS = Kp*17/16 + 1 slots apart, so the fill (lanes across rows), the LDS
// sort passes (lanes along a row) and the register blocks (a lane per 16
// consecutive keys) all hit distinct banks.
//
// Lane (g, s), s < S = NT / G, owns layers s, s + S, s + 2S, ... of pixel g.
// It loads their depth, alpha and colour together at the start of the group
// (the colours of its first kBigC layers wait in registers until the walk
// has produced the weights), so one memory round trip serves the group.
//
// Sort: bitonic, every comparator min-to-lower.  Comparators closer than 16
// positions never leave a 16-key block, so each block is sorted (sizes
// 2..16) or half-cleaned (strides 8..1 of every later merge) by one lane in
// registers.  The strides >= 16 of a merge go through LDS up to four at a
// time: a lane loads the 2^m keys that m consecutive stages compare only
// among themselves, runs the m stages in registers and writes the keys
// back, one barrier per pass.  For Kp = 512 that is 6 LDS passes, not 15.
// Positions K..Kp-1 hold the padding key, which no real key exceeds; as
// every comparator is min-to-lower they keep it throughout, so blocks and
// groups that lie wholly in the padding are skipped.
//
// The walk: the S lanes of a pixel take a product scan over S chunks of the
// sorted row; then colour sums in layer order and a fixed-order reduction
// over the S lanes.
#ifndef DFB_BLK_LOG
#define DFB_BLK_LOG 4
#endif
constexpr int kBlkLog = DFB_BLK_LOG;   // keys sorted per lane in registers: 2^kBlkLog
constexpr int kBlk = 1 << kBlkLog;
// Layers per lane whose colours are loaded with the keys (held in registers
// through the sort: 16 keeps the LDS-sort kernel at 247 VGPRs, 2 waves per
// SIMD, which its LDS allows anyway; 32 drops it to one), and the most merge
// stages one LDS pass runs.
#ifndef DFB_BIG_C
#define DFB_BIG_C 16
#endif
#ifndef DFB_MAX_M
#define DFB_MAX_M 4
#endif
// Layers per lane whose depth and alpha loads are in flight together past
// the first kBigC, and layers per lane whose colour loads are in flight
// together after the walk.  On the 8192^2 heavy-tailed frame, then sorted here
// whole, (16, 16, 8) took 34.4 ms against 35.7 ms for (8, 8, 4); larger
// batches of depth and alpha past the first 8 layers were slower (24, 24:
// 38.0-38.1 ms).
#ifndef DFB_BIG_FILL
#define DFB_BIG_FILL 16
#endif
#ifndef DFB_BIG_COLS
#define DFB_BIG_COLS 8
#endif
constexpr int kBigFill = DFB_BIG_FILL;
constexpr int kBigCols = DFB_BIG_COLS;
constexpr int kBigC = DFB_BIG_C;

__device__ __forceinline__ int kslot(int i) { return i + (i >> 4); }

// Plane loads of the LDS sort.
template <typename FT>
__device__ __forceinline__ float ldb(const FT* __restrict__ base, uint32_t i) {
#if DFB_BIGK_NT
  return ldf<FT>(base, i);
#else
  return static_cast<float>(base[i]);
#endif
}


// a block is read as runs of 16 keys, none of which straddles a pad slot
__device__ __forceinline__ void block_load(const uint64_t* r, int base, uint64_t (&k)[kBlk]) {
#pragma unroll
  for (int h = 0; h < kBlk / 16; ++h) {
    const uint64_t* q = r + kslot(base + 16 * h);
#pragma unroll
    for (int i = 0; i < 16; ++i) k[16 * h + i] = q[i];
  }
}
__device__ __forceinline__ void block_store(uint64_t* r, int base, const uint64_t (&k)[kBlk]) {
#pragma unroll
  for (int h = 0; h < kBlk / 16; ++h) {
    uint64_t* q = r + kslot(base + 16 * h);
#pragma unroll
    for (int i = 0; i < 16; ++i) q[i] = k[16 * h + i];
  }
}
// strides 8, 4, 2, 1 of a merge larger than the block (half-cleaners)
__device__ __forceinline__ void block_half_clean(uint64_t (&k)[kBlk]) {
#pragma unroll
  for (int str = kBlk / 2; str > 0; str >>= 1)
#pragma unroll
    for (int i = 0; i < kBlk; ++i)
      if ((i & str) == 0) KeyMinMax()(k[i], k[i + str]);
}

// One LDS pass over every row: M consecutive stages of the merge of size
// 2^ls, the first with stride 2^lt, the last with stride 2^lo (lo = lt-M+1).
// Group c of a row is the positions b + r 2^lo (r < 2^M), b being c with M
// zero bits inserted at lo..lt; these meet only each other in the M stages.
// When lt = ls - 1 the first stage is the merge's mirrored one (x against
// x ^ (2^ls - 1)) and the upper half of a group is the mirror image of its
// lower half, in increasing position order.
template <int M>
__device__ __forceinline__ void lds_stages(uint64_t* keys, int RS, int G, int lk, int ls, int lt,
                                           int K, int NT, int tid) {
  constexpr int N = 1 << M, H = N / 2, U = M >= 3 ? 1 : (M == 2 ? 2 : 4);  // groups in flight
  const int lo = lt - M + 1, glog = lk - M, total = G << glog;
  const bool mirror = lt == ls - 1;
  const int mask = (2 << lt) - 1;
  for (int e0 = tid; e0 < total; e0 += U * NT) {
    uint64_t v[U][N];
    int ix[U][N];
    bool act[U];
#pragma unroll
    for (int w = 0; w < U; ++w) {
      const int e = e0 + w * NT;
      const int g = e >> glog, c = e & ((1 << glog) - 1);
      const int b = ((c >> lo) << (lt + 1)) | (c & ((1 << lo) - 1));
      act[w] = e < total && b < K;  // b is the group's lowest position
#pragma unroll
      for (int r = 0; r < N; ++r) {
        const int pos = (mirror && r >= H) ? ((b + ((N - 1 - r) << lo)) ^ mask) : b + (r << lo);
        ix[w][r] = g * RS + kslot(pos);
        v[w][r] = act[w] ? keys[ix[w][r]] : kKeyPad;
      }
    }
#pragma unroll
    for (int w = 0; w < U; ++w) {
      if (mirror) {
#pragma unroll
        for (int r = 0; r < H; ++r) KeyMinMax()(v[w][r], v[w][N - 1 - r]);
      } else {
#pragma unroll
        for (int r = 0; r < H; ++r) KeyMinMax()(v[w][r], v[w][r + H]);
      }
#pragma unroll
      for (int k = M - 2; k >= 0; --k)
#pragma unroll
        for (int r = 0; r < N; ++r)
          if ((r & (1 << k)) == 0) KeyMinMax()(v[w][r], v[w][r | (1 << k)]);
      if (act[w]) {
#pragma unroll
        for (int r = 0; r < N; ++r) keys[ix[w][r]] = v[w][r];
      }
    }
  }
}

// G (pixels per group) for a padded layer count 2^lk and an LDS budget.
__device__ __forceinline__ int bigk_group(int lk, int budget, int NT) {
  const int RS = (1 << lk) + (1 << (lk - 4)) + 1;
  int G = budget / (RS * 12);
  G = G > NT ? NT : G;
  G = G > 64 ? 64 : G;
  while (G & (G - 1)) G &= G - 1;  // power of two
  return G;
}

template <typename FT>
__device__ float unit_bigk(const FrameArgs& a, const Unit& u, const int64_t* __restrict__ loff,
                           int K, int off, char* lds) {
  const int NT = blockDim.x, tid = threadIdx.x;
  const uint32_t P = static_cast<uint32_t>(a.P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  int lk = 6;                       // log2(Kp), Kp >= 64
  while ((1 << lk) < K) ++lk;
  const int Kp = 1 << lk;
  const int RS = Kp + (Kp >> 4) + 1;
  const int G = bigk_group(lk, a.big_lds, NT);
  int lg = 0;
  while ((1 << lg) < G) ++lg;
  const int S = NT / G;                   // lanes per pixel
  const int C = Kp / S > 0 ? Kp / S : 1;  // layers (and sorted positions) per lane
  uint64_t* keys = reinterpret_cast<uint64_t*>(lds);
  float* wv = reinterpret_cast<float*>(keys + static_cast<size_t>(G) * RS);
  float4* red = reinterpret_cast<float4*>(lds + a.big_lds);  // [NT]
  float* tend = reinterpret_cast<float*>(red + NT);           // [G], G <= 64
  int64_t* lofs = reinterpret_cast<int64_t*>(tend + 64);      // [K]
  for (int i = tid; i < K; i += NT) lofs[i] = loff[i];
  lds_barrier();
  const int gm = tid & (G - 1), sm = tid >> lg;
  const int nblk = G << (lk - kBlkLog);  // register blocks over all rows
  uint64_t* krow = keys + gm * RS;
  float* wrow = wv + gm * RS;
  float vs = 0.f;
  for (int q0 = 0; q0 < a.work_px; q0 += G) {
    const int qme = q0 + gm;
    const bool live = qme < a.work_px;
    bool in_me = false;
    const int p_me = live ? unit_pixel(a, u, qme, in_me) : 0;
    // 1. depth, alpha and colour of the lane's layers l = sm + j S, all
    //    loads issued before the first LDS store; padding keys sort last
    float cr[kBigC], cg[kBigC], cb[kBigC];
    {
      float dv[kBigC], av[kBigC];
#pragma unroll
      for (int j = 0; j < kBigC; ++j) {
        const int l = sm + j * S;
        dv[j] = 0.f;
        av[j] = 0.f;
        cr[j] = 0.f;
        cg[j] = 0.f;
        cb[j] = 0.f;
        if (j < C && live && l < K) {
          const FT* __restrict__ b = frag + lofs[l];
          dv[j] = ldb<FT>(b, 4 * P + p_me);
          av[j] = ldb<FT>(b, 3 * P + p_me);
        }
      }
#pragma unroll
      for (int j = 0; j < kBigC; ++j) {
        const int l = sm + j * S;
        if (j < C && live && l < K) {
          const FT* __restrict__ b = frag + lofs[l];
          cr[j] = ldb<FT>(b, p_me);
          cg[j] = ldb<FT>(b, P + p_me);
          cb[j] = ldb<FT>(b, 2 * P + p_me);
        }
      }
#pragma unroll
      for (int j = 0; j < kBigC; ++j) {
        const int l = sm + j * S;
        if (j < C) {
          krow[kslot(l)] = (live && l < K)
                               ? big_key(depth_bits(dv[j]), l) : kKeyPad;
          wrow[kslot(l)] = av[j];
        }
      }
    }
    for (int j0 = kBigC; j0 < C; j0 += kBigFill) {  // more layers than kBigC per lane: keys only here
      float dv[kBigFill], av[kBigFill];
#pragma unroll
      for (int j = 0; j < kBigFill; ++j) {
        const int l = sm + (j0 + j) * S;
        dv[j] = 0.f;
        av[j] = 0.f;
        if (j0 + j < C && live && l < K) {
          const FT* __restrict__ b = frag + lofs[l];
          dv[j] = ldb<FT>(b, 4 * P + p_me);
          av[j] = ldb<FT>(b, 3 * P + p_me);
        }
      }
#pragma unroll
      for (int j = 0; j < kBigFill; ++j) {
        const int l = sm + (j0 + j) * S;
        if (j0 + j < C) {
          krow[kslot(l)] = (live && l < K)
                               ? big_key(depth_bits(dv[j]), l) : kKeyPad;
          wrow[kslot(l)] = av[j];
        }
      }
    }
    lds_barrier();
    // 2. sort every row: blocks of 16 in registers first
    for (int b = tid; b < nblk; b += NT) {
      uint64_t k[kBlk];
      uint64_t* r = keys + (b >> (lk - kBlkLog)) * RS;
      const int base = (b & ((1 << (lk - kBlkLog)) - 1)) * kBlk;
      if (base < K) {
        block_load(r, base, k);
        sort_network<kBlk>(k, KeyMinMax());
        block_store(r, base, k);
      }
    }
    lds_barrier();
    for (int ls = kBlkLog + 1; ls <= lk; ++ls) {  // merge size 2^ls
      for (int lt = ls - 1; lt >= kBlkLog;) {     // strides >= kBlk through LDS
        const int m = lt - kBlkLog + 1 >= DFB_MAX_M ? DFB_MAX_M : lt - kBlkLog + 1;
        if (m == 4) lds_stages<4>(keys, RS, G, lk, ls, lt, K, NT, tid);
        else if (m == 3) lds_stages<3>(keys, RS, G, lk, ls, lt, K, NT, tid);
        else if (m == 2) lds_stages<2>(keys, RS, G, lk, ls, lt, K, NT, tid);
        else lds_stages<1>(keys, RS, G, lk, ls, lt, K, NT, tid);
        lt -= m;
        lds_barrier();
      }
      for (int b = tid; b < nblk; b += NT) {     // strides 8..1 in registers
        uint64_t k[kBlk];
        uint64_t* r = keys + (b >> (lk - kBlkLog)) * RS;
        const int base = (b & ((1 << (lk - kBlkLog)) - 1)) * kBlk;
        if (base < K) {
          block_load(r, base, k);
          block_half_clean(k);
          block_store(r, base, k);
        }
      }
      lds_barrier();
    }
    // 3. front-to-back walk: chunk products, exclusive scan over the S chunks.
    //    Rows past the unit's last pixel hold only padding keys: skipped.
    const int i0 = sm * C, i1 = live ? ((i0 + C < K) ? i0 + C : K) : 0;
    float prod = 1.f;
#pragma unroll 8
    for (int i = i0; i < i1; ++i) {
      const int l = key_layer(krow[kslot(i)]);
      prod = prod * (1.f - wrow[kslot(l)]);
    }
    red[tid].x = prod;
    lds_barrier();
    float T = 1.f;
    for (int s2 = 0; s2 < sm; ++s2) T = T * red[s2 * G + gm].x;
    lds_barrier();
    float Ap = 0.f;
#pragma unroll 4
    for (int i = i0; i < i1; ++i) {
      const int l = key_layer(krow[kslot(i)]);
      const float al = wrow[kslot(l)];
      wrow[kslot(l)] = T;
      Ap = fmaf(T, al, Ap);
      T = T * (1.f - al);
      if (a.mode & kModeKeepOrder)
        a.order[static_cast<size_t>(off + i) * P + p_me] = static_cast<uint16_t>(l);
    }
    lds_barrier();
    // 4. colour sums in layer order: T_l * c_l
    float R = 0.f, Gc = 0.f, B = 0.f;
    int sm4 = sm;
    asm volatile("" : "+v"(sm4));  // addresses are recomputed here, not kept across the sort
    if (live) {
#pragma unroll
      for (int j = 0; j < kBigC; ++j) {
        const int l = sm4 + j * S;
        if (j < C && l < K) {
          const float w = wrow[kslot(l)];
          R = fmaf(w, cr[j], R);
          Gc = fmaf(w, cg[j], Gc);
          B = fmaf(w, cb[j], B);
        }
      }
      int l = sm4 + kBigC * S;
      for (; l + (kBigCols - 1) * S < K; l += kBigCols * S) {
        float w[kBigCols], r4[kBigCols], g4[kBigCols], b4[kBigCols];
#pragma unroll
        for (int j = 0; j < kBigCols; ++j) {
          const FT* __restrict__ b = frag + lofs[l + j * S];
          w[j] = wrow[kslot(l + j * S)];
          r4[j] = ldb<FT>(b, p_me);
          g4[j] = ldb<FT>(b, P + p_me);
          b4[j] = ldb<FT>(b, 2 * P + p_me);
        }
#pragma unroll
        for (int j = 0; j < kBigCols; ++j) {
          R = fmaf(w[j], r4[j], R);
          Gc = fmaf(w[j], g4[j], Gc);
          B = fmaf(w[j], b4[j], B);
        }
      }
      for (; l < K; l += S) {
        const FT* __restrict__ b = frag + lofs[l];
        const float w = wrow[kslot(l)];
        R = fmaf(w, ldb<FT>(b, p_me), R);
        Gc = fmaf(w, ldb<FT>(b, P + p_me), Gc);
        B = fmaf(w, ldb<FT>(b, 2 * P + p_me), B);
      }
    }
    // lanes whose chunk is the last non-empty one hold the final T
    const int last = (K - 1) / C;
    red[tid] = make_float4(R, Gc, B, Ap);
    if (sm == last) tend[gm] = T;
    lds_barrier();
    if (sm == 0 && live) {
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int s2 = 0; s2 < S; ++s2) {
        const float4 v = red[s2 * G + gm];
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
      }
      vs += finish_px(a, u, p_me, in_me, with_background(a, u.t, p_me, acc, tend[gm]));
    }
    lds_barrier();
  }
  return vs;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ float variance_of_mean(float sum, int inside_px, int n) {
  if (n < 2) return __int_as_float(0x7f800000);
  return sum / (3.f * static_cast<float>(inside_px) * static_cast<float>(n) *
                static_cast<float>(n - 1));
}

// Work queue.  The work list is cut into blocks of B = queue_block
// consecutive positions (the units of one tile); counter s (of S = n_queues)
// holds the blocks congruent to s, in order.  Workgroup b starts on counter
// b mod S, and its first unit there is its rank r = b / S among those
// workgroups (no atomic).  Each ticket c of a counter names its unit g + c,
// g being the number of workgroups that start on it.  Lane 0 of wave 0
// takes the next ticket at the start of a unit and the result is read at
// its end, so the atomic's latency hides behind the unit's work.  A workgroup
// whose counter is drained reads all counters at once, one a lane, and goes
// on to the next open one (s + 1, s + 2, ... mod S) or ends.  A launch whose
// counters hold no more units than workgroups start on them (a.one_each)
// takes no tickets at all.  The row sort draws runs of consecutive units (run_of)
// and starts on one.  Workgroups are dealt to the 8 XCDs in turn and S
// is a multiple of 8 on every grid of 8 workgroups or more, so the units of
// one tile run at about the same time under one XCD's L2: unit rows that
// share cache lines (fp16 planes, units narrower than a line) are fetched
// from memory once.
struct Queue {
  uint32_t* ctr;
  int s, g, n;  // counter, workgroups starting on it, units it holds
  int run;      // units a workgroup starts with: the first g * run units are given without a ticket
};

// A draw of up to a.max_run consecutive units (the row sort's), fewer as the
// counter runs out: each workgroup's half share of what is left.
__device__ __forceinline__ int run_of(const FrameArgs& a, int left, int g) {
  const int n = left / (2 * g);
  return n < 1 ? 1 : (n < a.max_run ? n : a.max_run);
}

__device__ __forceinline__ Queue queue_of(const FrameArgs& a, int s) {
  Queue q;
  q.s = s;
  q.g = (static_cast<int>(gridDim.x) - s + a.n_queues - 1) / a.n_queues;
  q.n = queue_units(a.n_work, a.queue_block, a.n_queues, s);
  q.run = run_of(a, q.n, q.g);
  if (a.list_end < a.n_work) q.n = queue_units(a.list_end, a.queue_block, a.n_queues, s);
  q.ctr = a.queue + static_cast<size_t>(s) * kQueueStride + a.slot;
  return q;
}

// Work-list position of the j-th unit of a counter (j < q.n).
__device__ __forceinline__ int unit_at(const FrameArgs& a, const Queue& q, int j) {
  const int B = a.queue_block;
  return ((j / B) * a.n_queues + q.s) * B + j % B;
}

__device__ __forceinline__ uint32_t take_ticket(const Queue& q, int n = 1) {
  uint32_t v = 0;
  if (__lane_id() == 0) v = atomicAdd(q.ctr, static_cast<uint32_t>(n));
  return v;
}

// The index in its counter of the unit a ticket names, or -1: none left.
__device__ __forceinline__ int ticket_index(const Queue& q, uint32_t v) {
  const int64_t j = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(v)) + q.g * q.run;
  return j < q.n ? static_cast<int>(j) : -1;
}

// The next unit after counter q has no more for this launch (wave 0, all
// lanes): lane s reads counter s, so finding the open ones costs one trip to
// the coherent level and not one a counter.  `closed` holds the counters this
// workgroup is done with, so the loop ends.  Sets q to the unit's counter and
// count to the run drawn, and returns its first index there, or -1: the launch
// has no more.  Reading the
// counters in turn put 15 dependent trips behind the last unit of every
// workgroup; kernel times before, and now with the split finish counts and
// ticketless launches too: 256^2, 4 ranks 13.9 -> 7.1 us, 1280x720 27.4 -> 15.5,
// 1920x1080 fp16 average 25.4 -> 21.3, 4096x1024 fp16 159 -> 154 a frame.
__device__ __forceinline__ int next_open_unit(const FrameArgs& a, Queue& q, uint64_t& closed, int& count) {
  const int S = a.n_queues, lane = static_cast<int>(__lane_id());
  const Queue mine = queue_of(a, lane < S ? lane : 0);
  int j = -1;
  while (j < 0) {
    closed |= 1ull << q.s;
    const uint32_t c = __hip_atomic_load(mine.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t open = __ballot(lane < S && static_cast<int64_t>(c) + mine.g * mine.run < mine.n) & ~closed;
    if (open == 0) break;
    const uint64_t after = open & (~0ull << q.s);  // counters past q.s first, then from 0
    q = queue_of(a, __builtin_ctzll(after ? after : open));
    count = run_of(a, q.n - q.g * q.run - static_cast<int>(__builtin_amdgcn_readlane(c, q.s)), q.g);
    j = ticket_index(q, take_ticket(q, count));
  }
  return j;
}

// A unit's M2 sum (all waves) -> var_partial[w].  Runs on all lanes of wave
// 0; the combine into per-tile values is a separate kernel (no fences here).
__device__ __forceinline__ void store_partial(const FrameArgs& a, int w, const float* s_red,
                                              int n_waves) {
  float sum = 0.f;
  for (int i = 0; i < 4; ++i)
    if (i < n_waves) sum += s_red[i];
  if (__lane_id() == 0) a.var_partial[w] = sum;
}

// The persistent frame kernel.  Control flow that contains barriers is
// uniform across the workgroup; code that only lane 0 runs is a single
// store or atomic, so no lane can be left behind in a loop that holds a
// barrier.
#ifndef DFB_WAVES_F16_K32
#define DFB_WAVES_F16_K32 0
#endif
constexpr int min_waves(int kcap, bool half) {
  return kcap <= 8 ? (DFB_WAVES_K8 > 0 ? DFB_WAVES_K8 : 1)
                   : kcap <= 16 ? (DFB_WAVES_K16 > 0 ? DFB_WAVES_K16 : 1)
                                : (half && DFB_WAVES_F16_K32 > 0 ? DFB_WAVES_F16_K32
                                                                 : (DFB_WAVES_K32 > 0 ? DFB_WAVES_K32 : 1));
}

__device__ __forceinline__ FrameState* frame_state(const FrameArgs& a) { return a.state; }

// The frame's sequence number and accumulation count, read by every wave from
// the device state.  Nothing waits for them until they are used, so the
// unit's table reads run meanwhile.  The last workgroup to finish advances the
// state after every workgroup's wave 0 has counted it finished, so a read whose
// value is used has to come before its workgroup's count: a wave has its values
// before the barrier that ends its first unit.  Workgroup 0 recycles slots with
// every wave's value whether it has a unit or not; where it has none (a launch
// without units, every tile being deep) the host launches one wave, which reads
// before it counts.
__device__ __forceinline__ uint32_t read_frame_state(FrameArgs& a) {
  const FrameState* st = frame_state(a);
  const uint32_t seq = __hip_atomic_load(&st->seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  a.n_acc = __hip_atomic_load(&st->n_acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return seq;
}
__device__ __forceinline__ uint32_t use_frame_state(FrameArgs& a, uint32_t seq_in) {
  const uint32_t seq = __builtin_amdgcn_readfirstlane(seq_in);
  const int n_prev = static_cast<int>(__builtin_amdgcn_readfirstlane(a.n_acc));
  a.list_end = a.n_work;
  a.slot = static_cast<int32_t>(seq % kSlots);
  a.clear_slot = static_cast<int32_t>((seq + kSlots / 2) % kSlots);
  a.n_acc = (a.mode & kModeAccumulate) ? n_prev + 1 : n_prev;
  a.inv_n = a.n_acc > 0 ? 1.f / static_cast<float>(a.n_acc) : 1.f;
  return seq;
}

// Recycle the slot of the frame kSlots/2 ahead (counters, finish counts) in
// every ring.  The frame's last launch does it for all of them: a frame of
// another layer layout may not run the other launches, and a slot left
// uncleared would hand out no units kSlots frames later.
__device__ __forceinline__ void recycle_slots(const FrameArgs& a) {
  constexpr int kPages = kRings * (kQueues + 1);
  for (int i = threadIdx.x; i < 2 * kPages; i += blockDim.x)  // a page's ticket and finish counters
    __hip_atomic_store(a.rings + static_cast<size_t>(i % kPages) * kQueueStride + (i / kPages) * kFinishWord + a.clear_slot,
                       0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Count a workgroup finished (thread 0): among the workgroups of its home
// counter, and the last of those among the counters, so that no address takes
// more than grid / kQueues adds (an add to one address takes about 16 ns: 960
// workgroups that end together would queue for 15 us).  The last workgroup
// advances the frame state for the next frame (sequence number, and the
// accumulation count of an accumulating frame).  Every queue access of the
// workgroup has returned its value before this point.  Only the frame's last
// launch is counted.
__device__ __forceinline__ void finish_workgroup(const FrameArgs& a, uint32_t seq, int home) {
  const int tid = threadIdx.x;
  const int g = (static_cast<int>(gridDim.x) - home + a.n_queues - 1) / a.n_queues;
  uint32_t* mine = a.queue + static_cast<size_t>(home) * kQueueStride + kFinishWord + a.slot;
  uint32_t* all = a.queue + static_cast<size_t>(kQueues) * kQueueStride + kFinishWord + a.slot;
  uint32_t done = 0;
  if (tid == 0) done = __hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0 && done == static_cast<uint32_t>(g - 1)) {
    done = __hip_atomic_fetch_add(all, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (done == static_cast<uint32_t>(a.n_queues - 1)) {
      __hip_atomic_store(&frame_state(a)->seq, seq + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (a.mode & kModeAccumulate)
        __hip_atomic_store(&frame_state(a)->n_acc, a.n_acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The tile at a position of the launch's list; without a list, in tile order.
__device__ __forceinline__ TileRec tile_rec(const FrameArgs& a, const TileRec* __restrict__ recs,
                                            const int32_t* __restrict__ tile_off, int pos) {
  if (recs) return recs[pos];
  const int off = tile_off[pos];
  return {pos, off, tile_off[pos + 1] - off, 0};
}

// KCAP 8, 16, 32: register-sort capacity (tiles with more layers are other
// launches'); KCAP 0: only the tiles with more than a.big_min layers.
template <typename FT, int KCAP, int OP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(min_waves(KCAP, sizeof(FT) == 2))))
frame_kernel_t(FrameArgs args, const int32_t* __restrict__ tile_off,
               const int64_t* __restrict__ layer_off, const TileRec* __restrict__ recs) {
  extern __shared__ __align__(16) char lds[];
  // the next unit and a unit's M2 sums, in two buffers used in turn: a wave may
  // be a unit behind another, so one barrier a unit is enough
  __shared__ __align__(16) int4 s_next[2];
  __shared__ float s_red[2][4];
  constexpr bool kLast = KCAP > 0;  // the frame's last launch: it counts its workgroups and advances the state
  const int tid = threadIdx.x;
  const int n_waves = static_cast<int>(blockDim.x >> 6);
  const bool wave0 = __builtin_amdgcn_readfirstlane(tid) < 64;  // uniform per wave
  FrameArgs a = args;
  a.list_end = a.n_work;
  const uint32_t seq_read = read_frame_state(a);
  const int home = static_cast<int>(blockIdx.x) % a.n_queues;
  const int r = static_cast<int>(blockIdx.x) / a.n_queues;
  Queue q = queue_of(a, home);
  int it = r < q.n ? unit_at(a, q, r) : a.n_work;  // the first unit is static
  // its table entries are on their way while the state is read
  TileRec rec = {0, 0, 0, 0};
  if (it < a.n_work) rec = tile_rec(a, recs, tile_off, it / a.subs_per_tile);
  const uint32_t seq = use_frame_state(a, seq_read);
  q.ctr += a.slot;
  if (kLast && blockIdx.x == 0) recycle_slots(a);
  uint64_t closed = 0;  // counters this workgroup has found empty
  int turn = 0;
  while (it < a.n_work) {
    // the next unit's ticket is taken now and read after this unit's work
    const uint32_t next = wave0 && !a.one_each ? take_ticket(q) : 0u;
    Unit u;
    u.t = rec.tile;
    const int s = it - (it / a.subs_per_tile) * a.subs_per_tile, w = u.t * a.subs_per_tile + s;
    u.sy0 = (s / a.subs_x) * a.work_h;
    u.sx0 = (s - (s / a.subs_x) * a.subs_x) * a.work_w;
    u.y0 = (u.t / a.tiles_x) * a.tile_h;
    u.x0 = (u.t - (u.t / a.tiles_x) * a.tiles_x) * a.tile_w;
    const int off = rec.off, K = rec.layers;
    const int64_t* __restrict__ blk = layer_off + off;
    float* wl = reinterpret_cast<float*>(lds);
    float vs = 0.f;
    bool mine = true;  // uniform: this launch composites the unit
    if constexpr (KCAP == 0) {
      mine = K > a.big_min;
      if (mine) vs = unit_bigk<FT>(a, u, blk, K, off, lds);
    } else if constexpr (OP == DFB_OP_AVERAGE) {
      vs = (a.vec_ok && K > 0) ? unit_average_vec<FT>(a, u, blk, K) : unit_average<FT>(a, u, blk, K);
    } else if constexpr (OP == DFB_OP_LIST) {
      vs = K == 0 ? unit_background(a, u)
                  : (a.vec_ok ? unit_list_vec<FT>(a, u, blk, K, off) : unit_list<FT>(a, u, blk, K, off));
    } else {
    mine = K <= KCAP;
    if (K == 0) vs = unit_background(a, u);
    else if (K <= 1) vs = unit_reg<FT, 1, KCAP>(a, u, blk, K, off, wl);
    else if (K <= 2) vs = unit_reg<FT, 2, KCAP>(a, u, blk, K, off, wl);
    else if (K <= 3) vs = unit_reg<FT, 3, KCAP>(a, u, blk, K, off, wl);
    else if (K <= 4) vs = unit_reg<FT, 4, KCAP>(a, u, blk, K, off, wl);
    else if (K <= 6) vs = unit_reg<FT, 6, KCAP>(a, u, blk, K, off, wl);
    else if (K <= 8) vs = unit_reg<FT, 8, KCAP>(a, u, blk, K, off, wl);
    else if constexpr (KCAP >= 16) {
      // the kernel of a frame whose tiles have at most KCAP layers carries
      // no code for more: K <= KCAP here (the host picks KCAP >= the
      // frame's largest tile)
      if (K <= 12) vs = unit_reg<FT, 12, KCAP>(a, u, blk, K, off, wl);
      else if (KCAP == 16 || K <= 16) vs = unit_reg<FT, 16, KCAP>(a, u, blk, K, off, wl);
      else if constexpr (KCAP >= 32) {
        if (K <= 24) vs = unit_reg<FT, 24, KCAP>(a, u, blk, K, off, wl);
        else if (K <= 32) vs = unit_reg<FT, 32, KCAP>(a, u, blk, K, off, wl);
      }
    }
    }
    const bool acc = (a.mode & kModeAccumulate) != 0 && mine;
    if (acc) {
      vs = wave_sum(vs);  // fixed-order reductions only: deterministic
      if ((tid & 63) == 0) s_red[turn][tid >> 6] = vs;
    }
    if (wave0 && !a.one_each) {  // the next unit and its tile, while the other waves finish this one
      int j = ticket_index(q, next);
      int one = 1;
      if (j < 0) j = next_open_unit(a, q, closed, one);
      const int v = j < 0 ? a.n_work : unit_at(a, q, j);
      int4 n = {v, 0, 0, 0};
      if (v < a.n_work) {
        const TileRec t = tile_rec(a, recs, tile_off, v / a.subs_per_tile);
        n = {v, t.tile, t.off, t.layers};
      }
      if (__lane_id() == 0) s_next[turn] = n;
    }
    lds_barrier();  // s_red and s_next complete
    if (wave0 && acc) store_partial(a, w, s_red[turn], n_waves);
    if (a.one_each) break;
    const int4 n = s_next[turn];
    it = __builtin_amdgcn_readfirstlane(n.x);
    rec = {__builtin_amdgcn_readfirstlane(n.y), __builtin_amdgcn_readfirstlane(n.z), __builtin_amdgcn_readfirstlane(n.w), 0};
    turn ^= 1;
  }
  if (kLast) finish_workgroup(a, seq, home);
}

// ------------------------------------------------- 32 < K <= 512: row sort
// A workgroup of 8 waves takes groups of 32 consecutive pixels of a tile (one
// 128-byte line of an fp32 plane per layer); each wave sorts 4 of them, 16
// lanes a pixel, in registers (rowsort.h).
//   1. depth and alpha rows are loaded, 4 pixels a lane; the depths go through
//      the LDS array rows[layer][32 pixels] to the lanes that sort them, then
//      the alphas take their place
//   2. the row sort
//   3. the walk: each lane reads its positions' alphas by layer, the lanes'
//      products are scanned over the row, and the transmittance in front of
//      every layer replaces its alpha
//   4. colour rows are loaded and weighted, summed over a lane's layers, over
//      the lanes and waves of a pixel in a fixed order
// Every sum is split the same way whatever the launch shape is.
//
// Bound by vector instructions: 106 a key, padding keys among them (87 in the
// sort), at 81 % of the issue slots on the 8192^2 frame below (fp16, 1500x1100:
// 70 %); 20 bytes a fragment (fp32) are two thirds of what memory moves in that
// time.  The LDS sort it replaces for these counts was bound by the latency of
// its passes at 8 waves a compute unit, and read each 128-byte line twice.
// 8192^2 heavy-tailed frame (57.9 GB, up to 512 layers): 36.9 -> 13.4 ms a frame;
// 1500x1100 fp16, up to 128 layers: 504 -> 150 us.
// Rows are 36 words apart: the 16 lanes of a pixel (at consecutive layers)
// and the wave's 4 pixels hit all 64 banks once.
constexpr int kDeepPitch = 36;
constexpr int kDeepWaves = kDeepThreads / 64;
constexpr int kDeepRows = kDeepThreads / 8;  // layers loaded per pass: 8 lanes of 4 pixels each
__host__ __device__ constexpr size_t deep_rows_bytes(int max_layers) {  // one row more: the padding keys' alpha 0
  return static_cast<size_t>(max_layers + 1) * kDeepPitch * sizeof(float);
}
// after the rows and the layer offsets: the waves' colour sums, then the
// final transmittance and alpha of every pixel
constexpr size_t kDeepTail = (kDeepWaves * 3 + 2) * kDeepPx * sizeof(float);

// 4 consecutive elements of a plane as they lie in memory.
template <typename FT>
struct Quad;
template <>
struct Quad<float> {
  typedef float V __attribute__((ext_vector_type(4)));
  using RK = RowKey64;
  static __device__ __forceinline__ float4 f(V v) { return make_float4(v.x, v.y, v.z, v.w); }
  static __device__ __forceinline__ uint4 bits(V v) { return __builtin_bit_cast(uint4, v); }
  // Ordered depth bits << 17 | the byte offset of the layer's pixel in the LDS
  // rows, below the exponent of 2^52 (a normal double, as big_key): the walk
  // needs no multiplication.  `flip` reverses the key (its sign).
  static __device__ __forceinline__ uint64_t key(uint32_t bits, int l, int px, uint32_t flip) {
    const float d = __uint_as_float(bits) + 0.f;  // -0 -> +0
    const uint32_t b = __float_as_uint(d), s = static_cast<uint32_t>(static_cast<int32_t>(b) >> 31) | 0x80000000u;
    const uint32_t x = d != d ? 0xFFFFFFFFu : b ^ s;
    return (static_cast<uint64_t>(__builtin_amdgcn_alignbit(0x2198u | (flip >> 17), x, 15)) << 32) | (x << 17) |
           static_cast<uint32_t>((l * kDeepPitch + px) * 4);
  }
  static constexpr uint32_t kNaN = 0x7FC00000u;
  static __device__ __forceinline__ int at(uint64_t k, int) { return static_cast<int>(static_cast<uint32_t>(k) & 0x1FFFFu); }
};
template <>
struct Quad<_Float16> {
  typedef _Float16 V __attribute__((ext_vector_type(4)));
  using RK = RowKey32;
  static __device__ __forceinline__ float4 f(V v) {
    return make_float4(static_cast<float>(v.x), static_cast<float>(v.y), static_cast<float>(v.z), static_cast<float>(v.w));
  }
  static __device__ __forceinline__ uint4 bits(V v) {
    const uint2 u = __builtin_bit_cast(uint2, v);
    return make_uint4(u.x & 0xFFFFu, u.x >> 16, u.y & 0xFFFFu, u.y >> 16);
  }
  // Ordered depth bits << 13 | the layer's row of 144 bytes in steps of 16
  static __device__ __forceinline__ int32_t key(uint32_t bits, int l, int, uint32_t) {
    return static_cast<int32_t>(half_depth_bits(static_cast<uint16_t>(bits)) << 13) | (l * (kDeepPitch / 4));
  }
  static constexpr uint32_t kNaN = 0x7E00u;
  static __device__ __forceinline__ int at(int32_t k, int px_bytes) { return ((k & 0x1FFF) << 4) + px_bytes; }
};

// Pixels p .. p + 3 of a plane (aligned: the host checked P % 4 and the base).
template <typename FT>
__device__ __forceinline__ typename Quad<FT>::V load_quad(const FT* __restrict__ plane, int p) {
  return __builtin_nontemporal_load(reinterpret_cast<const typename Quad<FT>::V*>(plane + p));
}

// x + the value of the lane 16 (32) lanes away, in both.
__device__ __forceinline__ float add_xor16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor8(float x) {
  return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, true));  // row_ror:8
}

// Pixels [p0, p1) of tile u.t, K <= 16 R layers; every group's M2 sum goes to
// a.deep_partial.
template <typename FT, int R, int RMAX>
__device__ __forceinline__ void deep_unit(const FrameArgs& a, const Unit& u, int K_in, int off, int p0, int p1, float* rows,
                                           const int64_t* lofs, float* red) {
  using Q = Quad<FT>;
  using V = typename Q::V;
  using RK = typename Q::RK;
  constexpr int NP = (16 * R + kDeepRows - 1) / kDeepRows;  // passes over the layers
  constexpr int NC = NP % 4 == 0 ? 4 : (NP % 3 == 0 ? 3 : NP);  // passes whose colours are in flight together
  static_assert(NP % NC == 0, "colour batches");
  // Up to 128 layers the registers hold a group's colours across the sort and
  // the next group's depths and alphas behind it, so that every load of a group
  // is under way while another phase computes (8192^2: 12.7 -> 12.2 ms, 1500x1100
  // fp16: 112 -> 108 us); not in the fp32 kernels held to 80 registers, where
  // they would spill.
  constexpr bool EARLY = NP <= 2 && (sizeof(FT) == 2 || RMAX >= 32);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, j = lane & 15, rank = RK::rank(j), px = wave * 4 + (lane >> 4);
  const int quad0 = (tid & 7) * 4;
  const int P = a.P;
  const size_t plane = static_cast<size_t>(P);
  const FT* __restrict__ frag = static_cast<const FT*>(a.frag);
  float* tend = red + kDeepWaves * 3 * kDeepPx;
  float* asum = tend + kDeepPx;
  // Opaque copies, made anew in every group and phase: the addresses and
  // the l < K masks of a phase are computed there and not kept in registers
  // across the sort.
  int K = K_in, row0 = tid >> 3;
  V dv[NP], av[NP], cv[NC][3];
  auto load_depth_alpha = [&](int pq) {
#pragma unroll
    for (int i = 0; i < NP; ++i) dv[i] = load_quad<FT>(frag + lofs[min(row0 + i * kDeepRows, K - 1)] + 4 * plane, pq);
#pragma unroll
    for (int i = 0; i < NP; ++i) av[i] = load_quad<FT>(frag + lofs[min(row0 + i * kDeepRows, K - 1)] + 3 * plane, pq);
  };
  auto load_colours = [&](int i0, int pq) {  // of passes i0 .. i0 + NC - 1
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      asm volatile("" : "+s"(K));
      const FT* __restrict__ b = frag + lofs[min(row0 + (i0 + i) * kDeepRows, K - 1)];
#pragma unroll
      for (int c = 0; c < 3; ++c) cv[i][c] = load_quad<FT>(b + c * plane, pq);
    }
  };
  // past the end of a tile whose last group is ragged: its last pixels again
  if constexpr (EARLY) load_depth_alpha(p0 + quad0 < P ? p0 + quad0 : P - 4);
  for (int g0 = p0; g0 < p1; g0 += kDeepPx) {
    const int pq = g0 + quad0 < P ? g0 + quad0 : P - 4;
    K = K_in;
    row0 = tid >> 3;
    asm volatile("" : "+s"(K), "+v"(row0));
    // 1. depth and alpha rows
    if constexpr (!EARLY) load_depth_alpha(pq);
    if constexpr (EARLY) load_colours(0, pq);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int l = min(row0 + i * kDeepRows, K - 1);
      *reinterpret_cast<uint4*>(rows + l * kDeepPitch + quad0) = Q::bits(dv[i]);
    }
    // row K: a NaN depth and alpha 0 for the padding keys, which sort last
    if (tid < 8) *reinterpret_cast<uint4*>(rows + K * kDeepPitch + quad0) = make_uint4(Q::kNaN, Q::kNaN, Q::kNaN, Q::kNaN);
    lds_barrier();
    int jl = j;
    const uint32_t flip = rank & 1 ? 0x80000000u : 0u;
    asm volatile("" : "+s"(K), "+v"(jl));
    typename RK::K key[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r && r % 8 == 0) __builtin_amdgcn_sched_barrier(0);  // reads of 8 keys at a time: registers
      const int l = min(r * 16 + jl, K);
      key[r] = Q::key(__float_as_uint(rows[l * kDeepPitch + px]), l, px, flip);
    }
    lds_barrier();
    asm volatile("" : "+s"(K), "+v"(row0));
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int l = min(row0 + i * kDeepRows, K - 1);
      *reinterpret_cast<float4*>(rows + l * kDeepPitch + quad0) = Q::f(av[i]);
    }
    if (tid < 8) *reinterpret_cast<float4*>(rows + K * kDeepPitch + quad0) = make_float4(0.f, 0.f, 0.f, 0.f);
    if (EARLY && g0 + kDeepPx < p1) load_depth_alpha(g0 + kDeepPx + quad0 < P ? g0 + kDeepPx + quad0 : P - 4);
    // 2. sort
    __builtin_amdgcn_sched_barrier(0);
    row_sort<RK, R>(key, lane);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    // 3. walk
    asm volatile("" : "+s"(K), "+v"(row0));
    const int p_me = g0 + px;
    if ((a.mode & kModeKeepOrder) && p_me < P) {
      int i0 = rank * R;
      asm volatile("" : "+v"(i0));
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (i0 + r < K)
          a.order[static_cast<size_t>(off + i0 + r) * P + p_me] = static_cast<uint16_t>(Q::at(key[r], 0) / (kDeepPitch * 4));
    }
    int at[R];
    float al[R];
    float prod = 1.f;
    char* column = reinterpret_cast<char*>(rows);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      at[r] = Q::at(key[r], px * 4);
      al[r] = *reinterpret_cast<float*>(column + at[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) prod *= 1.f - al[r];
    float T = row_product_before<RK>(prod), A = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      *reinterpret_cast<float*>(column + at[r]) = T;
      A = fmaf(T, al[r], A);
      T *= 1.f - al[r];
    }
    A = row_sum(A);
    if (rank == 15) {
      tend[px] = T;
      asum[px] = A;
    }
    lds_barrier();
    // 4. colours
    float acc[3][4];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[c][v] = 0.f;
#pragma unroll
    for (int i0 = 0; i0 < NP; i0 += NC) {
      if constexpr (!EARLY) load_colours(i0, pq);
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int l = row0 + (i0 + i) * kDeepRows;
        if (l < K) {
          const float4 w = *reinterpret_cast<const float4*>(rows + l * kDeepPitch + quad0);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float4 x = Q::f(cv[i][c]);
            acc[c][0] = fmaf(w.x, x.x, acc[c][0]);
            acc[c][1] = fmaf(w.y, x.y, acc[c][1]);
            acc[c][2] = fmaf(w.z, x.z, acc[c][2]);
            acc[c][3] = fmaf(w.w, x.w, acc[c][3]);
          }
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[c][v] = add_xor32(add_xor16(add_xor8(acc[c][v])));
    if (lane < 8) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
        *reinterpret_cast<float4*>(red + (wave * 3 + c) * kDeepPx + quad0) =
            make_float4(acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
    }
    lds_barrier();
    float vs = 0.f;
    if (tid < kDeepPx && g0 + tid < p1) {
      float s[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kDeepWaves; ++w)
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += red[(w * 3 + c) * kDeepPx + tid];
      const int p = g0 + tid, ty = p / a.tile_w, tx = p - ty * a.tile_w;
      const bool inside = u.x0 + tx < a.width && u.y0 + ty < a.height;
      vs = finish_px(a, u, p, inside, with_background(a, u.t, p, make_float4(s[0], s[1], s[2], asum[tid]), tend[tid]));
    }
    if ((a.mode & kModeAccumulate) && wave == 0) {
      vs = wave_sum(vs);
      if (lane == 0) a.deep_partial[static_cast<size_t>(u.t) * a.deep_subs + g0 / kDeepPx] = vs;
    }
  }
}

// Waves per SIMD the register allocation is held to: 512 layers need 74 KB of
// LDS a workgroup, so two of 8 waves fit a compute unit; up to 256, three, with
// 80 registers a lane.  In the kernel of up to 256 layers that spills 36 in fp32 and 13
// in fp16.  Against 4 waves and 128 registers, 64 tiles of 64x64 with 130 / 192 / 256
// layers take 211 / 243 / 317 us for 213 / 243 / 301 in fp32 and 182 / 212 / 270 for
// 195 / 219 / 275 in fp16; 256 tiles of 100 to 256 layers 913 for 899 and 731 for 778.
constexpr int deep_waves(int rmax) { return rmax >= 32 ? 4 : 6; }

// RMAX: keys per lane, 16 RMAX layers at most.
template <typename FT, int RMAX>
__global__ void __launch_bounds__(kDeepThreads) __attribute__((amdgpu_waves_per_eu(deep_waves(RMAX))))
deep_kernel_t(FrameArgs args, const int32_t* __restrict__ tile_off, const int64_t* __restrict__ layer_off,
              const TileRec* __restrict__ recs) {
  extern __shared__ __align__(16) char lds[];
  __shared__ __align__(16) int4 s_next;
  const int tid = threadIdx.x;
  const bool wave0 = __builtin_amdgcn_readfirstlane(tid) < 64;  // uniform per wave
  FrameArgs a = args;
  use_frame_state(a, read_frame_state(a));
  // the rows first: their offset is a constant that the LDS instructions carry
  float* rows = reinterpret_cast<float*>(lds);
  int64_t* lofs = reinterpret_cast<int64_t*>(lds + deep_rows_bytes(a.deep_layers));
  float* red = reinterpret_cast<float*>(lofs + a.deep_layers);
  // A unit is one group of kDeepPx pixels; a workgroup draws runs of them.
  const int home = static_cast<int>(blockIdx.x) % a.n_queues;
  Queue q = queue_of(a, home);
  uint64_t closed = 0;
  int j = static_cast<int>(blockIdx.x) / a.n_queues * q.run, count = q.run;  // the run: units j .. j + count - 1 of q
  if (j >= q.n) return;
  for (;;) {
    count = count < q.n - j ? count : q.n - j;
    const int count_next = run_of(a, q.n - j - count, q.g);
    const uint32_t next = wave0 && !a.one_each ? take_ticket(q, count_next) : 0u;
    bool mine = true;
    while (count > 0 && mine) {  // in two where a run goes over the end of a block or of a tile
      const int it = unit_at(a, q, j), pos = it / a.deep_subs, piece = it - pos * a.deep_subs;
      const int n = min(count, min(a.deep_subs - piece, a.queue_block - j % a.queue_block));
      const TileRec rec = tile_rec(a, recs, tile_off, pos);
      Unit u;
      u.t = rec.tile;
      u.sx0 = u.sy0 = 0;
      u.y0 = (u.t / a.tiles_x) * a.tile_h;
      u.x0 = (u.t - (u.t / a.tiles_x) * a.tiles_x) * a.tile_w;
      const int off = rec.off, K = rec.layers;
      mine = K > kRegMax;
      // the list is in descending order of layers: a tile of few ends it, for
      // every counter (asking each in turn took 15 draws of every workgroup)
      if (!mine) a.list_end = min(a.list_end, pos * a.deep_subs);
      if (mine && K <= kDeepMax && K <= a.deep_layers) {
        for (int i = tid; i < K; i += kDeepThreads) lofs[i] = layer_off[off + i];
        lds_barrier();
        const int p0 = piece * kDeepPx, p1 = p0 + n * kDeepPx < a.P ? p0 + n * kDeepPx : a.P;
        if (K <= 64) deep_unit<FT, 4, RMAX>(a, u, K, off, p0, p1, rows, lofs, red);
        else if (K <= 96) deep_unit<FT, 6, RMAX>(a, u, K, off, p0, p1, rows, lofs, red);
        else if (RMAX == 8 || K <= 128) deep_unit<FT, 8, RMAX>(a, u, K, off, p0, p1, rows, lofs, red);
        else if constexpr (RMAX >= 16) {
          if (K <= 192) deep_unit<FT, 12, RMAX>(a, u, K, off, p0, p1, rows, lofs, red);
          else if (RMAX == 16 || K <= 256) deep_unit<FT, 16, RMAX>(a, u, K, off, p0, p1, rows, lofs, red);
          else if constexpr (RMAX >= 32) {
            if (K <= 384) deep_unit<FT, 24, RMAX>(a, u, K, off, p0, p1, rows, lofs, red);
            else deep_unit<FT, 32, RMAX>(a, u, K, off, p0, p1, rows, lofs, red);
          }
        }
      }
      j += n;
      count -= n;
      lds_barrier();  // the LDS rows and offsets are free; every lane has read s_next
    }
    if (a.one_each) break;
    if (wave0) {
      int jn = mine ? ticket_index(q, next) : -1, cn = count_next;
      if (jn < 0) jn = next_open_unit(a, q, closed, cn);
      if (__lane_id() == 0) s_next = {jn, cn, q.s, 0};
    }
    lds_barrier();
    const int4 sn = s_next;
    j = __builtin_amdgcn_readfirstlane(sn.x);
    if (j < 0) break;
    count = __builtin_amdgcn_readfirstlane(sn.y);
    const int counter = __builtin_amdgcn_readfirstlane(sn.z);
    if (counter != q.s) q = queue_of(a, counter);  // wave 0 is there already
  }
}

// Per-tile variance of the mean from the units' partial M2 sums, added in
// unit order (deterministic): one thread per tile.
__global__ void __launch_bounds__(256) tile_variance_kernel_t(VarianceArgs a) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= a.n_tiles) return;
  const float* __restrict__ part = a.var_partial + t * a.subs_per_tile;
  int n = a.subs_per_tile;
  if (a.deep_subs) {  // the tile was composited by the row-sort launch, in units of its own
    const int K = a.tile_off[t + 1] - a.tile_off[t];
    if (K > kRegMax && K <= kDeepMax) {
      part = a.deep_partial + t * a.deep_subs;
      n = a.deep_subs;
    }
  }
  float sum = 0.f;
  for (int i = 0; i < n; ++i) sum += part[i];
  const int x0 = (t % a.tiles_x) * a.tile_w, y0 = (t / a.tiles_x) * a.tile_h;
  const int wx = a.width - x0, wy = a.height - y0;
  const int inside = (wx < a.tile_w ? wx : a.tile_w) * (wy < a.tile_h ? wy : a.tile_h);
  a.tile_var[t] = variance_of_mean(sum, inside, a.state->n_acc);
}

// Unfused accumulation of the stored finished tiles: one workgroup per tile.
__global__ void __launch_bounds__(256) accumulate_kernel_t(AccumArgs a) {
  __shared__ float s_red[4];
  const int t = blockIdx.x, tid = threadIdx.x;
  const int n_acc = a.state->n_acc + 1;  // the state kernel after this launch advances it
  const float inv_n = 1.f / static_cast<float>(n_acc);
  const int x0 = (t % a.tiles_x) * a.tile_w, y0 = (t / a.tiles_x) * a.tile_h;
  float vs = 0.f;
  for (int p = tid; p < a.P; p += blockDim.x) {
    const int py = p / a.tile_w, pxl = p - py * a.tile_w;
    const bool inside = (x0 + pxl < a.width) && (y0 + py < a.height);
    const size_t px = static_cast<size_t>(t) * a.P + p;
    const float4 x = reinterpret_cast<const float4*>(a.finished)[px];
    vs += store_pixel(x, px, static_cast<size_t>(t) * 3 * a.P + p, a.P, inside,
                      (a.mode & ~kModeKeepFinished) | kModeAccumulate, n_acc, inv_n,
                      a.inv_gamma, nullptr, a.accum, a.m2, a.final_out);
  }
  vs = wave_sum(vs);
  if ((tid & 63) == 0) s_red[tid >> 6] = vs;
  lds_barrier();
  if (__builtin_amdgcn_readfirstlane(tid) < 64) {
    const int n_waves = static_cast<int>(blockDim.x >> 6);
    float sum = 0.f;
    for (int i = 0; i < 4; ++i)
      if (i < n_waves) sum += s_red[i];
    const int wx = a.width - x0, wy = a.height - y0;
    const int inside = (wx < a.tile_w ? wx : a.tile_w) * (wy < a.tile_h ? wy : a.tile_h);
    if (__lane_id() == 0) a.tile_var[t] = variance_of_mean(sum, inside, n_acc);
  }
}

// Accumulation count of a handle's frame state, set (value >= 0) or advanced
// by one (value < 0), stream-ordered with the frames around it.
__global__ void state_kernel_t(FrameState* st, int32_t value) {
  if (threadIdx.x == 0 && blockIdx.x == 0) st->n_acc = value >= 0 ? value : st->n_acc + 1;
}

// n words of p set to v (grid-stride).
__global__ void fill_u32_kernel_t(uint32_t* __restrict__ p, uint32_t v, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = v;
}

// n words copied (grid-stride); src may be pinned host memory.
__global__ void copy_u32_kernel_t(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    dst[i] = src[i];
}

// Longest-first list of the tiles on the device, from the per-tile CSR offsets:
// a counting sort by layer count, descending (one workgroup of kLptThreads
// lanes; equal counts in any order, which changes only the order units are
// taken in, never a result).
constexpr int kLptBins = kMaxLayers + 1;                                // K = 0 .. kMaxLayers
constexpr int kLptPer = (kLptBins + kLptThreads - 1) / kLptThreads;    // bins per lane in the scan
__global__ void __launch_bounds__(kLptThreads) lpt_work_kernel_t(const int32_t* __restrict__ tile_off,
                                                                 int32_t n_tiles, TileRec* __restrict__ recs) {
  __shared__ int32_t cnt[kLptBins];     // bin j holds layer count K = kMaxLayers - j
  __shared__ int32_t wave_tot[kLptThreads / 64];
  const int tid = threadIdx.x;
  for (int j = tid; j < kLptBins; j += kLptThreads) cnt[j] = 0;
  __syncthreads();
  for (int t = tid; t < n_tiles; t += kLptThreads) {
    int K = tile_off[t + 1] - tile_off[t];
    K = K < 0 ? 0 : (K > kMaxLayers ? kMaxLayers : K);
    atomicAdd(&cnt[kMaxLayers - K], 1);
  }
  __syncthreads();
  // exclusive scan of the bins: each lane sums kLptPer consecutive bins,
  // the lane sums are scanned within waves and across the waves
  int local[kLptPer];
  int sum = 0;
#pragma unroll
  for (int i = 0; i < kLptPer; ++i) {
    const int j = tid * kLptPer + i;
    local[i] = j < kLptBins ? cnt[j] : 0;
    sum += local[i];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if ((tid & 63) >= o) incl += v;
  }
  if ((tid & 63) == 63) wave_tot[tid >> 6] = incl;
  __syncthreads();
  int base = 0;
  for (int w = 0; w < (tid >> 6); ++w) base += wave_tot[w];
  int run = base + incl - sum;   // exclusive prefix of this lane's first bin
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kLptPer; ++i) {
    const int j = tid * kLptPer + i;
    if (j < kLptBins) cnt[j] = run;
    run += local[i];
  }
  __syncthreads();
  for (int t = tid; t < n_tiles; t += kLptThreads) {
    const int off = tile_off[t], layers = tile_off[t + 1] - off;
    const int K = layers < 0 ? 0 : (layers > kMaxLayers ? kMaxLayers : layers);
    recs[atomicAdd(&cnt[kMaxLayers - K], 1)] = {t, off, layers, 0};
  }
}

// NaN scan of every layer's depth plane: one workgroup per layer.
template <typename FT>
__global__ void __launch_bounds__(256) validate_kernel_t(ValidateArgs a) {
  const int l = blockIdx.x;
  if (l >= a.n_layers) return;
  const FT* __restrict__ b = static_cast<const FT*>(a.frag) + a.layer_off[l];
  bool bad = false;
  for (int p = threadIdx.x; p < a.P; p += blockDim.x) {
    const float d = ldf<FT>(b, 4 * static_cast<uint32_t>(a.P) + p);
    bad |= (d != d);
  }
  if (bad) atomicOr(a.bad, 1u);
}

}  // namespace

const void* frame_kernel(int dtype, int kcap, int op) {
  if (kcap == 0)
    return dtype == 0 ? reinterpret_cast<const void*>(&frame_kernel_t<float, 0, 0>)
                      : reinterpret_cast<const void*>(&frame_kernel_t<_Float16, 0, 0>);
  if (dtype == 0) {
    if (op == DFB_OP_LIST) return reinterpret_cast<const void*>(&frame_kernel_t<float, 8, DFB_OP_LIST>);
    if (op == DFB_OP_AVERAGE) return reinterpret_cast<const void*>(&frame_kernel_t<float, 8, DFB_OP_AVERAGE>);
    if (kcap <= 8) return reinterpret_cast<const void*>(&frame_kernel_t<float, 8, 0>);
    if (kcap <= 16) return reinterpret_cast<const void*>(&frame_kernel_t<float, 16, 0>);
    return reinterpret_cast<const void*>(&frame_kernel_t<float, 32, 0>);
  }
  if (op == DFB_OP_LIST) return reinterpret_cast<const void*>(&frame_kernel_t<_Float16, 8, DFB_OP_LIST>);
  if (op == DFB_OP_AVERAGE) return reinterpret_cast<const void*>(&frame_kernel_t<_Float16, 8, DFB_OP_AVERAGE>);
  if (kcap <= 8) return reinterpret_cast<const void*>(&frame_kernel_t<_Float16, 8, 0>);
  if (kcap <= 16) return reinterpret_cast<const void*>(&frame_kernel_t<_Float16, 16, 0>);
  return reinterpret_cast<const void*>(&frame_kernel_t<_Float16, 32, 0>);
}

const void* deep_kernel(int dtype, int max_layers) {
  if (dtype == 0) {
    if (max_layers <= 128) return reinterpret_cast<const void*>(&deep_kernel_t<float, 8>);
    if (max_layers <= 256) return reinterpret_cast<const void*>(&deep_kernel_t<float, 16>);
    return reinterpret_cast<const void*>(&deep_kernel_t<float, 32>);
  }
  if (max_layers <= 128) return reinterpret_cast<const void*>(&deep_kernel_t<_Float16, 8>);
  if (max_layers <= 256) return reinterpret_cast<const void*>(&deep_kernel_t<_Float16, 16>);
  return reinterpret_cast<const void*>(&deep_kernel_t<_Float16, 32>);
}

size_t deep_lds_bytes(int max_layers) {
  const int k = deep_layers(max_layers);
  return kDeepTail + k * sizeof(int64_t) + deep_rows_bytes(k);
}

const void* accumulate_kernel() { return reinterpret_cast<const void*>(&accumulate_kernel_t); }

const void* tile_variance_kernel() { return reinterpret_cast<const void*>(&tile_variance_kernel_t); }

const void* state_kernel() { return reinterpret_cast<const void*>(&state_kernel_t); }

const void* fill_u32_kernel() { return reinterpret_cast<const void*>(&fill_u32_kernel_t); }

const void* copy_u32_kernel() { return reinterpret_cast<const void*>(&copy_u32_kernel_t); }

const void* lpt_work_kernel() { return reinterpret_cast<const void*>(&lpt_work_kernel_t); }

const void* validate_kernel(int dtype) {
  return dtype == 0 ? reinterpret_cast<const void*>(&validate_kernel_t<float>)
                    : reinterpret_cast<const void*>(&validate_kernel_t<_Float16>);
}

int big_lds_bytes(int max_layers) {
  // 16 pixels per group at 512 padded layers needs 16 * 545 * 12 bytes
  return max_layers > 256 ? kBigLdsBytes : (max_layers > 128 ? 96 * 1024 : 64 * 1024);
}

size_t frame_lds_bytes(int kcap, int threads, int max_layers, int big_lds) {
  if (kcap > 0) return static_cast<size_t>(kcap) * threads * sizeof(float);  // the walk's alpha / T columns
  // keys + alpha, the reduction rows [threads] float4, T_end [64], layer offsets [max_layers]
  return big_lds + static_cast<size_t>(threads) * 16 + 64 * 4 + static_cast<size_t>(max_layers) * 8;
}

}  // namespace dfb
