// gfx950 kernels of the denoiser: BF16 MFMA implicit-GEMM conv3x3 forward,
// data gradient and weight gradient (FP32 accumulation), and the small
// elementwise / reduction kernels around them.  Every reduction has a fixed
// order (partials per chunk, then a sequential sum), so results are
// deterministic.
//
// The three convolutions are one GEMM shape, D[M][N] += A[M][K] B[K][N],
// read from LDS in K slices:
//   forward  M = c_out,  N = pixels, K = (tap, c_in)   A = W, B = x[p + tap]
//   dgrad    M = c_in,   N = pixels, K = (tap, c_out)  A = W^T, B = dy[p - tap]
//   wgrad    M = c_in,   N = c_out, K = pixels (per tap, split over chunks)
// All three use v_mfma_f32_32x32x16_bf16.  Operand layout (checked on the
// device): lane l holds k = (l/32)*8 .. +7 of row/column l%32; the result
// element r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "dfb_internal.h"
#include "unet_internal.h"

namespace dfb {
namespace unet {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t to_bf16(float f) {  // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

// ------------------------------------------------------------- forward
// Persistent implicit-GEMM conv3x3 forward.  A workgroup computes TH x
// 32-pixel output tiles (each XCD has one band of them, handed out in order)
// for all BN output channels; a tile is CP/32 steps, one per
// 32-input-channel slice.  A step stages the slice's input halo ((TH+2) x 34
// pixels, zero outside the image; with UP the (TH/2+2) x 18 source pixels the
// up-sampled halo reads) and, unless all slices' weights stay resident, the
// slice's weights of all nine taps in LDS, then runs the nine taps' MFMAs
// with no barrier between them.  The next step's halo and weights are loaded
// into registers while this step's MFMAs run, so a workgroup hides its own
// load latency.
//
// The MFMA is v_mfma_f32_32x32x16_bf16 (measured on the device: about 2.0
// PFLOP/s, against about 1.15 for v_mfma_f32_16x16x32_bf16 with the same
// number of independent accumulators).  It takes the weights as its row
// operand (32 output channels) and a 32-pixel tile row as its column
// operand; lane l holds pixel l % 32 and, in accumulator element r, channel
// 8 (r / 4) + 4 (l / 32) + r % 4.  A workgroup is CS * TH/2 waves; each
// owns two tile rows and BN / CS output channels (CS = 2 for 128 channels,
// else 1), so a taller tile spreads a staged weight slice over more waves at
// the same registers per wave.  The accumulators start from the bias;
// the epilogue (ReLU, v_cvt_pk_bf16_f32, optionally the 2x2 average pool, or
// instead of the stores the network's output conv written into a
// compositor frame) goes through a staging tile in LDS so that the stores
// are coalesced.
//
// LDS rows hold 32 bf16 channels (4 16-byte chunks).  gfx950 serves a
// ds_read_b128 16 lanes per cycle (per half-wave, the lanes whose bits 2-4
// have even parity, then odd), and a fragment read is 32 consecutive rows
// at one chunk per half-wave.  Halo pixels are 5 chunks apart (an odd pitch
// puts each 16-lane set on distinct banks wherever the 32 pixels start);
// weight rows are 4 chunks apart with the chunk index XOR-ed with
// (row >> 2) & 3, which does the same for 32 rows starting at a multiple of
// 32 (measured on the device: conflicting patterns take 2x the cycles).
// Every address of the tap loop is a per-lane register plus an immediate,
// so the loop issues no vector ALU work.
constexpr int kTW = 32;  // tile width (pixels)
constexpr int kXcds = 8;  // XCDs (each with its own L2) the workgroups of a launch are dealt to in turn
constexpr int kKC = 32;  // input channels per step
constexpr int kTicketStride = kTicketWords / kXcds;  // a counter of its own line for each XCD
// Output-tile heights (rows of 32 pixels, 8 or 16) of the layers with
// (output, input) channels (32, 32), (32, 64), (64, 32), (64, 64), (64, 128)
// and (128, *).  16 rows (8 waves) for the 64-channel layers: a staged
// weight slice serves twice the pixels (2048^2 enc2b / dec2b 107 / 98 -> 94 /
// 87 us, dec2a 181 -> 169 us); and for the 32 -> 32 layers (4 waves per
// SIMD instead of 3: enc1b 131 -> 126 us).  The 32 -> 64 and 64 -> 32
// layers were slower with 16 rows (dec1a 186 -> 199, enc2a 53 -> 56 us) and
// the 128-channel ones would spill.
#ifndef DFB_TH_32_32
#define DFB_TH_32_32 16
#endif
#ifndef DFB_TH_32_64
#define DFB_TH_32_64 8
#endif
#ifndef DFB_TH_64_32
#define DFB_TH_64_32 8
#endif
#ifndef DFB_TH_64_64
#define DFB_TH_64_64 16
#endif
#ifndef DFB_TH_64_128
#define DFB_TH_64_128 16
#endif
#ifndef DFB_TH_128
#define DFB_TH_128 8
#endif
// the same for the up-sampled layers (32, 64) and (64, 128)
#ifndef DFB_THU_32_64
#define DFB_THU_32_64 8
#endif
#ifndef DFB_THU_64_128
#define DFB_THU_64_128 16
#endif

// Waves that share a tile's 128 output channels (each takes 128 / DFB_CS_128
// of them): 2 halves the accumulators per wave, so the 128-channel layers
// run 2 waves per SIMD instead of 1 at the same LDS.
#ifndef DFB_CS_128
#define DFB_CS_128 2
#endif
// LDS bytes up to which a layer keeps every input slice's weights resident
// (the 16-row 64 -> 64 layers need 123 KB: one 8-wave workgroup per CU)
#ifndef DFB_RESW_KB
#define DFB_RESW_KB 124
#endif
template <int BN, int TH, int NCH, bool UP>
struct ConvCfg {
  // With UP the halo is staged at the source resolution: (TH/2 + 2) x 18
  // pixels, each read by the up to four output-halo pixels it is
  // up-sampled to (the fragment reads index it through the same
  // nearest-neighbour map).
  static constexpr int SHH = UP ? TH / 2 + 2 : TH + 2, SHW = UP ? kTW / 2 + 2 : kTW + 2;  // staged rows, columns
  static constexpr int HPITCH = 5;             // 16-byte chunks per halo pixel (4 used)
  static constexpr int HALO_CH = SHH * SHW * HPITCH;  // 16-byte chunks of a step's halo
  static constexpr int HALO_EL = SHH * SHW * 4;       // chunks loaded per step
  static constexpr int W_CH = 9 * BN * 4;      // 16-byte chunks of a step's weights
  static constexpr int CS = BN >= 128 ? DFB_CS_128 : 1;  // waves sharing a tile row pair's channels
  static constexpr int NT = 32 * TH * CS;      // threads: CS waves per two tile rows
  static constexpr int HIT = (HALO_EL + NT - 1) / NT, WIT = (W_CH + NT - 1) / NT;
  // The epilogue's staging tile (TH x 32 pixels of BN bf16 + 8 padding)
  // overlays the halo region, and the weights when a step re-stages them;
  // it is written in two passes of TH/2 rows when it does not fit.  The
  // small halo of an up-sampled layer is given room for at least one pass
  // (counting the weights' region when even the halo alone leaves no room
  // for all weight slices).
  static constexpr int STG1 = TH * kTW * (BN + 8) * 2;  // bytes of the whole staging tile
  static constexpr int WEXTRA = NCH > 1 && (HALO_CH + NCH * W_CH) * 16 + BN * 4 > DFB_RESW_KB * 1024 ? W_CH : 0;
  static constexpr int REGION_CH = UP && (HALO_CH + WEXTRA) * 16 < STG1 / 2 ? STG1 / 32 - WEXTRA : HALO_CH;
  // weight slices held in LDS: all of them when the layer's LDS stays
  // within DFB_RESW_KB (no weight traffic per step), else the step's slice,
  // re-staged every step
  static constexpr int WS = (REGION_CH + NCH * W_CH) * 16 + BN * 4 <= DFB_RESW_KB * 1024 ? NCH : 1;
  static constexpr int STG_ROOM = (WS == 1 && NCH > 1 ? REGION_CH + W_CH : REGION_CH) * 16;
  static constexpr int NPASS = STG1 <= STG_ROOM ? 1 : 2;
  static constexpr size_t BYTES = static_cast<size_t>(REGION_CH + WS * W_CH) * 16 + BN * 4;  // + the bias
  // waves per SIMD the register allocation is held to: those of the
  // workgroups that fit a compute unit's 160 KB of LDS, at most 4
  static constexpr int LDS_WG = static_cast<int>((160 * 1024) / BYTES);
  // ... and at most 2 where a step re-stages 64 or more channels' weights:
  // their prefetch registers and accumulators need more than 168 VGPRs
  static constexpr int REG_WAVES = WS == 1 && NCH > 1 && BN >= 64 ? 2 : 4;
  static constexpr int WAVES_LDS = LDS_WG * NT / 256 < 1 ? 1 : (LDS_WG * NT / 256 > 4 ? 4 : LDS_WG * NT / 256);
  static constexpr int WAVES = WAVES_LDS < REG_WAVES ? WAVES_LDS : REG_WAVES;
};
// Raw buffer accesses with a 2 GB range from a per-step base: an offset of
// kOOB is out of range, so the load returns zeros or the store is dropped.
// Every lane issues every access, so the number of outstanding memory
// operations is known at compile time and waiting for the prefetched loads
// never waits for the stores issued after them.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kOOB = static_cast<int>(0x80000000u);
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7FFFFFFF, 0x00020000);
}
__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t r, int byte_off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, 0);
  return uint4{v[0], v[1], v[2], v[3]};
}
// Cache policy of a store: kNT marks it non-temporal (streamed past the
// caches).  The first layer and the 32 -> 64 and 64 -> 128 layers store
// their activations that way (2048^2: enc1a 64 -> 55, dec1a 184 -> 176,
// dec2a 170 -> 165 us); the 32 -> 32 layers were slower with it (enc1b 125
// -> 130, dec1b 105 -> 113 us) and the others unchanged.
constexpr int kNT = 2;
template <int POLICY = 0>
__device__ __forceinline__ void buf_store16(__amdgpu_buffer_rsrc_t r, int byte_off, uint4 v) {
  const u32x4 w = {v.x, v.y, v.z, v.w};
  __builtin_amdgcn_raw_buffer_store_b128(w, r, byte_off, 0, POLICY);
}
__device__ __forceinline__ void buf_store8(__amdgpu_buffer_rsrc_t r, int byte_off, uint32_t lo, uint32_t hi) {
  const u32x2 v = {lo, hi};
  __builtin_amdgcn_raw_buffer_store_b64(v, r, byte_off, 0, 0);
}
// LDS chunk of (row p, chunk q) of the swizzled weights
__device__ __forceinline__ int swz(int p, int q) { return p * 4 + (q ^ ((p >> 2) & 3)); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// two floats to bf16 (round to nearest even), packed low | high << 16
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }


// Epilogue kinds: plain, plus the 2x2 average pool, or instead of storing
// y the network's 1x1 output conv and residual written straight into a
// compositor frame (inference, 32 channels).
enum Epi { kEpiPlain = 0, kEpiPool = 1, kEpiFrame = 2 };
struct OutConv {     // out[p][c] = mean[p][c] + b[c] + sum_i y[p][i] w[i][c], c < 3
  const float* w;    // [32][3]
  const float* b;    // [3]
  // the frame's running mean (tile-major) and tile variances: pixel e of the
  // frame becomes den[e] = (out[p], mean alpha), or the mean itself where
  // the tile falls back (n >= 2 and its variance above tau)
  FrameGlue glue;
  float tau;
  float* den;        // [T][P][4]
};

template <int BN, int CP, int TH, bool UP, int EPI>
__global__ void __launch_bounds__((ConvCfg<BN, TH, CP / kKC, UP>::NT))
__attribute__((amdgpu_waves_per_eu(ConvCfg<BN, TH, CP / kKC, UP>::WAVES)))
conv_fwd_k(Map x, Map x2, const uint16_t* __restrict__ w, const float* __restrict__ bias, Map y, Map pool, OutConv oc,
           Shape s, uint32_t* __restrict__ tickets) {
  __shared__ int s_next;
  using C = ConvCfg<BN, TH, CP / kKC, UP>;
  constexpr bool POOL = EPI == kEpiPool, OUT = EPI == kEpiFrame;
  constexpr int STORE_POLICY = (BN == 32 && CP == 64) || (BN == 64 && CP == 128) ? kNT : 0;
  static_assert(!OUT || BN == 32, "the output conv takes 32 channels, one pixel per thread");
  constexpr int NT = C::NT;  // threads (CS waves per two tile rows)
  constexpr int NCH = CP / kKC, MB = 2, NB = BN / 32 / C::CS;  // tile rows and 32-channel blocks per wave
  static_assert(NB >= 1 && NB * 32 * C::CS == BN, "channel split");
  constexpr int SHH = C::SHH, SHW = C::SHW, HALO_EL = C::HALO_EL, HIT = C::HIT, WIT = C::WIT;
  static_assert(!POOL || MB % 2 == 0, "the pool pairs rows inside a wave");
  extern __shared__ __align__(16) uint4 lds4[];
  uint4* halo = lds4;                // [SHH * SHW][5], and the epilogue's staging tile
  uint4* wts = lds4 + C::REGION_CH;  // [WS][9 * BN][4]
  float* lbias = reinterpret_cast<float*>(wts + C::WS * C::W_CH);  // [BN]: read per tile through LDS, so
  // starting a tile waits on no global load issued after the prefetch
  float* lout = lbias + BN;  // [32 * 3 + 3] output-conv weights and bias (kEpiFrame)
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  // wave = (channel group) * TH/2 + (row pair): rows 2 rw, 2 rw + 1 and the
  // channel blocks cb0 / 32 .. + NB - 1
  const int rw = C::CS > 1 ? wave % (TH / 2) : wave, cb0 = C::CS > 1 ? (wave / (TH / 2)) * NB * 32 : 0;
  const int tiles_x = (s.w + kTW - 1) / kTW, tiles_y = (s.h + TH - 1) / TH;
  const long long tiles = static_cast<long long>(s.n) * tiles_x * tiles_y;
  // The hardware deals workgroups to the 8 XCDs in turn.  XCD x, with n_x of
  // the G workgroups, has one contiguous band of tiles in row order, so the
  // workgroups on neighbouring tiles share their halos through one L2.  In
  // the band, workgroup xr takes tiles xr and n_x + xr, then the tiles its
  // tickets give: workgroups of a compute unit do not advance alike (the
  // oldest is served first: with equal shares of tiles, up1 of a 2048^2 frame
  // ended after 85 to 153 us in its 768 workgroups), and those ahead take
  // more (up1 128 -> 123 us; 8x256x512 forward 409 -> 399).  What bounds the
  // layers with 64 and more channels is the matrix cores at the clock they
  // sustain: without any load or store up1 takes 112 us; fragments read two or
  // three steps ahead, or fewer of them, change nothing.
  const long long G = gridDim.x;
  const int xcd = static_cast<int>(blockIdx.x % kXcds), xr = static_cast<int>(blockIdx.x / kXcds);
  const int n_x = static_cast<int>(G / kXcds) + (xcd < G % kXcds);
  const long long b0 = xcd * (G / kXcds) + (xcd < G % kXcds ? xcd : G % kXcds);
  const int t_first = static_cast<int>(b0 * tiles / G), band = static_cast<int>((b0 + n_x) * tiles / G) - t_first;
  const bool ticketed = band > 2 * n_x;  // uniform
  const int hi = UP ? s.h / 2 : s.h, wi = UP ? s.w / 2 : s.w;  // the map x is read from
  // The input is the channel concatenation of x and x2 (x2.c may be 0; else
  // x.c is a multiple of 32 and x2.ld == x.ld): slices below x.c read x, the
  // others x2.
  const int cin = x.c + x2.c;
  const bool full = cin == CP;  // else channels cin .. CP-1 are staged as zeros
  struct Tile {
    int n, ty, tx;
  };
  auto decode = [&](int i) {  // tile i of the band
    Tile u;
    const int t = t_first + i, per_img = tiles_x * tiles_y;
    u.n = t / per_img;
    const int r = t - u.n * per_img;
    u.ty = r / tiles_x;
    u.tx = r - u.ty * tiles_x;
    return u;
  };

  // this thread's halo elements e = tid + NT k: halo pixel e / 4 (row, column),
  // chunk e % 4; byte offset from the step's source origin (the halo's
  // top-left pixel, or the pixel it is up-sampled from); LDS chunk
  // hlds + 64 * HPITCH * k
  int hrel[HIT];
#pragma unroll
  for (int k = 0; k < HIT; ++k) {
    const int e = tid + NT * k, hp = e >> 2, cc = e & 3, hr = hp / SHW, hc = hp - hr * SHW;
    hrel[k] = e < HALO_EL ? ((hr * wi + hc) * x.ld + cc * 8) * 2 : kOOB;
  }
  const int hlds = (tid >> 2) * C::HPITCH + (tid & 3);
  // fragment reads of 16-channel half kh: weights of (tap, j) at
  // wts[(tap * BN + j * 32) * 4 + boff[kh]], halo of (m, tap) at
  // halo[aoff[dc] + hrow(m + dr) * SHW * HPITCH + 2 kh], where output-halo
  // row r of the wave is staged row r (or (r + 1) / 2 with UP) and
  // aoff[dc] holds the lane's column: l32 + dc (or (l32 + dc + 1) / 2)
  const int boff[2] = {l32 * 4 + ((0 + lh) ^ ((l32 >> 2) & 3)), l32 * 4 + ((2 + lh) ^ ((l32 >> 2) & 3))};
  const int wrow0 = UP ? rw * MB / 2 : rw * MB;  // the wave's first staged row (MB is even with UP)
  int aoff[UP ? 3 : 1];
#pragma unroll
  for (int dc = 0; dc < (UP ? 3 : 1); ++dc)
    aoff[dc] = (wrow0 * SHW + (UP ? (l32 + dc + 1) >> 1 : l32)) * C::HPITCH + lh;

  // Halo of slice ck of tile u into hreg; every load is issued (with
  // `none`, all out of range).
  auto load_halo = [&](const Tile& u, int ck, bool none, uint4* hreg) {
    const int oy0 = u.ty * TH, ox0 = u.tx * kTW;
    const bool second = ck * kKC >= x.c;
    const Map& xm = second ? x2 : x;
    const int cb = second ? ck * kKC - x.c : ck * kKC;  // first channel of the slice in xm
    const uint16_t* img = xm.p + xm.off + cb + static_cast<long long>(u.n) * hi * wi * xm.ld;
    // the staged halo's top-left pixel in the map read (hi x wi)
    const int sy0 = UP ? oy0 / 2 - 1 : oy0 - 1, sx0 = UP ? ox0 / 2 - 1 : ox0 - 1;
    const bool inner = full && sy0 >= 0 && sy0 + SHH <= hi && sx0 >= 0 && sx0 + SHW <= wi;
    const __amdgpu_buffer_rsrc_t src = buf_rsrc(img + (static_cast<long long>(sy0) * wi + sx0) * x.ld);
    int off[HIT];
    if (inner && !none) {
#pragma unroll
      for (int k = 0; k < HIT; ++k) off[k] = hrel[k];
    } else {  // zeros outside the image and past xm.c
#pragma unroll
      for (int k = 0; k < HIT; ++k) {
        const int e = tid + NT * k, hp = e >> 2, cc = e & 3, hr = hp / SHW, hc = hp - hr * SHW;
        const int r = sy0 + hr, c = sx0 + hc;
        const int ok = (static_cast<unsigned>(r) < static_cast<unsigned>(hi)) &
                       (static_cast<unsigned>(c) < static_cast<unsigned>(wi)) & (cb + cc * 8 < xm.c) & !none;
        off[k] = ok ? hrel[k] : kOOB;
      }
    }
#pragma unroll
    for (int k = 0; k < HIT; ++k) hreg[k] = buf_load16(src, off[k]);
  };
  // weights [tap][co][cin]: a step's slice is 64 bytes of each (tap, co) row
  const __amdgpu_buffer_rsrc_t wsrc = buf_rsrc(w);
  int wrel[WIT];  // byte offset of this thread's chunks in slice 0
#pragma unroll
  for (int k = 0; k < WIT; ++k) {
    const int e = tid + NT * k;
    wrel[k] = e < C::W_CH ? ((e >> 2) * cin + (e & 3) * 8) * 2 : kOOB;
  }
  auto load_w = [&](int ck, bool none, uint4* wreg) {
    int off[WIT];
    if (full && !none) {
#pragma unroll
      for (int k = 0; k < WIT; ++k) off[k] = wrel[k] + ck * kKC * 2;  // kOOB stays out of range
    } else {
#pragma unroll
      for (int k = 0; k < WIT; ++k) {
        const int cc = (tid + NT * k) & 3;
        off[k] = !none && ck * kKC + cc * 8 < cin ? wrel[k] + ck * kKC * 2 : kOOB;
      }
    }
#pragma unroll
    for (int k = 0; k < WIT; ++k) wreg[k] = buf_load16(wsrc, off[k]);
  };
  auto store_w = [&](const uint4* wreg, int slot) {
#pragma unroll
    for (int k = 0; k < WIT; ++k) {
      const int e = tid + NT * k;
      if (e < C::W_CH) wts[slot * C::W_CH + swz(e >> 2, e & 3)] = wreg[k];
    }
  };
  f32x16 acc[MB][NB];
  // Epilogue of tile u: ReLU and bf16 into a staging tile in LDS (over the
  // halo, and over the weights when a step re-stages them), then 16-byte
  // stores with consecutive lanes on consecutive addresses, and the 2x2
  // pool from the staging tile.  Output channels j*32 + 8q + 4*lh .. +3 of
  // pixel l32 are accumulator elements 4q .. 4q+3.  When the staging tile
  // does not fit it is written and stored in two passes of TH/2 rows.  With
  // `dummy` only the global stores are issued, all out of range: the
  // prologue issues the same stores as a loop iteration, so the loop entry
  // and its back edge leave the same memory operations behind the prefetch
  // and the wait for it is exact on both.
  constexpr int LDO = BN + 8;  // staging row (one pixel) in bf16
  constexpr int OCH = BN / 8;  // 16-byte chunks per output pixel
  constexpr int NPASS = C::NPASS;
  constexpr int RP = TH / NPASS;  // tile rows per pass
  static_assert(RP * kTW * LDO * 2 <= C::STG_ROOM, "staging tile too large");
  static_assert((RP * kTW * OCH) % NT == 0 && RP % 2 == 0 && RP % MB == 0, "pass shape");
  static_assert(!OUT || NPASS == 1, "the output conv reads every staged row of the tile");
  constexpr int NOUT = OUT ? 0 : RP * kTW * OCH / NT;                             // stores per thread and pass
  constexpr int NPOOL = POOL ? ((RP / 2) * (kTW / 2) * OCH + NT - 1) / NT : 0;  // pool stores per thread and pass
  uint16_t* stg = reinterpret_cast<uint16_t*>(lds4);
  // kEpiFrame: the mean RGBA and tile variance of this thread's pixel of the
  // tile being computed, and its frame index
  float bcur[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
  int ecur = 0;
  const int n_acc = OUT ? oc.glue.state->n_acc : 0;
  auto epilogue = [&](const Tile& u, bool dummy) {
    const int n = u.n, oy0 = u.ty * TH, ox0 = u.tx * kTW;
    const bool out_full = oy0 + TH <= s.h && ox0 + kTW <= s.w;
    const __amdgpu_buffer_rsrc_t yb = buf_rsrc(y.p + y.off + ((static_cast<long long>(n) * s.h + oy0) * s.w + ox0) * y.ld);
    const int ph = s.h / 2, pw = s.w / 2;
    const __amdgpu_buffer_rsrc_t pb =
        buf_rsrc(POOL ? pool.p + pool.off + ((static_cast<long long>(n) * ph + oy0 / 2) * pw + ox0 / 2) * pool.ld : y.p);
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
      if (!dummy) {
        __syncthreads();  // every wave is done with the halo / weights (or the previous pass)
        if (rw * MB / RP == pass) {
#pragma unroll
          for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const f32x16& v = acc[m][j];
                const int lrow = rw * MB + m - pass * RP;
                *reinterpret_cast<uint2*>(stg + (lrow * kTW + l32) * LDO + cb0 + j * 32 + 8 * q + 4 * lh) =
                    uint2{pack_bf16(fmaxf(v[4 * q], 0.f), fmaxf(v[4 * q + 1], 0.f)),
                          pack_bf16(fmaxf(v[4 * q + 2], 0.f), fmaxf(v[4 * q + 3], 0.f))};
              }
        }
        __syncthreads();
      }
#pragma unroll
      for (int k = 0; k < NOUT; ++k) {
        const int e = tid + NT * k, px = e / OCH, c = e % OCH, lrow = px / kTW, col = px % kTW;
        const int row = pass * RP + lrow;
        const int ok = !dummy & (out_full | ((oy0 + row < s.h) & (ox0 + col < s.w)));
        const uint4 v = dummy ? uint4{0u, 0u, 0u, 0u} : *reinterpret_cast<const uint4*>(stg + (lrow * kTW + col) * LDO + c * 8);
        // (distinct out-of-range offsets: identical ones would let the compiler drop all but the last)
        buf_store16<STORE_POLICY>(yb, ok ? ((row * s.w + col) * y.ld + c * 8) * 2 : kOOB + (pass * NOUT + k) * 16, v);
      }
#pragma unroll
      for (int k = 0; k < NPOOL; ++k) {
        // pooled pixel (qr, qc) of this pass: ((a + b) + c) + d of the staged
        // bf16 values, a b over c d
        const int e = tid + NT * k, qi = e / OCH, c = e % OCH, qr = qi / (kTW / 2), qc = qi % (kTW / 2);
        const int prow = pass * RP / 2 + qr;
        const int ok = !dummy & (e < (RP / 2) * (kTW / 2) * OCH) &
                       (out_full | ((oy0 / 2 + prow < ph) & (ox0 / 2 + qc < pw)));
        uint4 o = {0u, 0u, 0u, 0u};
        if (!dummy && e < (RP / 2) * (kTW / 2) * OCH) {
          const uint16_t* t00 = stg + ((2 * qr) * kTW + 2 * qc) * LDO + c * 8;
          const uint4 a4 = *reinterpret_cast<const uint4*>(t00);
          const uint4 b4 = *reinterpret_cast<const uint4*>(t00 + LDO);
          const uint4 c4 = *reinterpret_cast<const uint4*>(t00 + kTW * LDO);
          const uint4 d4 = *reinterpret_cast<const uint4*>(t00 + (kTW + 1) * LDO);
          const uint32_t A[4] = {a4.x, a4.y, a4.z, a4.w}, B[4] = {b4.x, b4.y, b4.z, b4.w},
                         Cc[4] = {c4.x, c4.y, c4.z, c4.w}, D[4] = {d4.x, d4.y, d4.z, d4.w};
          uint32_t r4[4];
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            const float lo = ((bf16_lo(A[h]) + bf16_lo(B[h])) + bf16_lo(Cc[h])) + bf16_lo(D[h]);
            const float hi2 = ((bf16_hi(A[h]) + bf16_hi(B[h])) + bf16_hi(Cc[h])) + bf16_hi(D[h]);
            r4[h] = pack_bf16(0.25f * lo, 0.25f * hi2);
          }
          o = uint4{r4[0], r4[1], r4[2], r4[3]};
        }
        buf_store16(pb, ok ? ((prow * pw + qc) * pool.ld + c * 8) * 2 : kOOB + (NPASS * NOUT + pass * NPOOL + k) * 16, o);
      }
      if (OUT) {
        // pixel tid of the tile: the 1x1 conv over its 32 staged bf16
        // channels, in channel order, then (mean + b) + sum
        const int lrow = tid / kTW, col = tid % kTW, row = pass * RP + lrow;
        const int ok = !dummy & (out_full | ((oy0 + row < s.h) & (ox0 + col < s.w)));
        float o3[3] = {0.f, 0.f, 0.f};
        if (!dummy) {
          float a3[3] = {0.f, 0.f, 0.f};
#pragma unroll
          for (int c8 = 0; c8 < 4; ++c8) {
            const uint4 v = *reinterpret_cast<const uint4*>(stg + (lrow * kTW + col) * LDO + c8 * 8);
            const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int i = c8 * 8 + k;
              const float xi = (k & 1) ? bf16_hi(wv[k >> 1]) : bf16_lo(wv[k >> 1]);
#pragma unroll
              for (int c = 0; c < 3; ++c) a3[c] = fmaf(xi, lout[i * 3 + c], a3[c]);
            }
          }
#pragma unroll
          for (int c = 0; c < 3; ++c) o3[c] = (bcur[c] + lout[96 + c]) + a3[c];
        }
        const bool fb = n_acc >= 2 && bcur[4] > oc.tau;
        const u32x4 dv = {__float_as_uint(fb ? bcur[0] : o3[0]), __float_as_uint(fb ? bcur[1] : o3[1]),
                          __float_as_uint(fb ? bcur[2] : o3[2]), __float_as_uint(bcur[3])};
        __builtin_amdgcn_raw_buffer_store_b128(dv, buf_rsrc(oc.den), ok ? ecur * 16 : kOOB + pass * 16, 0, 0);
      }
    }
  };

  uint4 hreg[HIT], wreg[WIT];
  float breg[5] = {0.f, 0.f, 0.f, 0.f, 0.f};  // bcur and ecur of the tile being prefetched
  int ereg = 0;
  auto load_base = [&](const Tile& u, bool none) {
    if (!OUT) return;
    const int oy0 = u.ty * TH, ox0 = u.tx * kTW, row = tid / kTW, col = tid % kTW;
    const FrameGlue& g = oc.glue;
    const int r = oy0 + row, c = ox0 + col, ty = r / g.tile_h, tx = c / g.tile_w, t = ty * g.tiles_x + tx;
    const int ok = !none & (r < s.h) & (c < s.w);
    ereg = t * g.P + (r - ty * g.tile_h) * g.tile_w + (c - tx * g.tile_w);
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(buf_rsrc(g.accum), ok ? ereg * 16 : kOOB, 0, 0);
    const uint32_t var = __builtin_amdgcn_raw_buffer_load_b32(buf_rsrc(g.tile_var), ok ? t * 4 : kOOB, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) breg[i] = __uint_as_float(v[i]);
    breg[4] = __uint_as_float(var);
  };
  if (tid < BN) lbias[tid] = bias[tid];
  if (OUT && tid < 99) lout[tid] = tid < 96 ? oc.w[tid] : oc.b[tid - 96];
  int i_nxt = xr + n_x;              // the next tile; from band on: none
  Tile cur = decode(xr), nxt = cur;  // the tile computed, the tile prefetched (G <= tiles: band >= n_x)
  constexpr bool RESW = C::WS == NCH;  // every slice's weights stay in LDS for every tile
  if (RESW) {
#pragma unroll
    for (int ck = 0; ck < NCH; ++ck) {
      load_w(ck, false, wreg);
      store_w(wreg, ck);
    }
  }
  load_halo(nxt, 0, false, hreg);
  if (!RESW) load_w(0, false, wreg);
  load_base(nxt, false);
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][j][r] = 0.f;
  epilogue(cur, true);
  for (;;) {
    const bool last = i_nxt >= band;
    uint32_t ticket = 0;
#pragma unroll
    for (int ck = 0; ck < NCH; ++ck) {
      __syncthreads();  // the previous step's fragment reads are done
#pragma unroll
      for (int k = 0; k < HIT; ++k)
        if (tid + NT * k < HALO_EL) halo[hlds + (NT / 4) * C::HPITCH * k] = hreg[k];
      if (!RESW) store_w(wreg, 0);
      if (OUT && ck == 0) {
#pragma unroll
        for (int i = 0; i < 5; ++i) bcur[i] = breg[i];
        ecur = ereg;
      }
      __syncthreads();
      // the tile after the next, asked for ahead of the loads that are waited
      // for before it is needed
      if (ck == 0 && ticketed && !last && tid == 0)
        ticket = __hip_atomic_fetch_add(tickets + xcd * kTicketStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // prefetch the next step: the next slice, or slice 0 of the next tile
      const bool none = ck == NCH - 1 && last;
      if (ck == NCH - 1 && !none) nxt = decode(i_nxt);
      load_halo(nxt, (ck + 1) % NCH, none, hreg);
      if (!RESW) load_w((ck + 1) % NCH, none, wreg);
      if (ck == NCH - 1) load_base(nxt, none);
      // keep the prefetch ahead of the taps: the scheduler would otherwise
      // sink the loads below the MFMAs and expose their latency
      __builtin_amdgcn_sched_barrier(0);
      if (ck == 0) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 b4 = *reinterpret_cast<const f32x4*>(lbias + cb0 + j * 32 + 8 * q + 4 * lh);
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[m][j][4 * q + r] = b4[r];
          }
      }
      // 18 (tap, 16-channel half) steps; the fragments of step i + 1 are
      // read while step i's MFMAs run
      bf16x8 wf[2][NB], hf[2][MB];
      auto frag = [&](int i, int bsel) {
        const int tap = i >> 1, kh = i & 1, dr = tap / 3, dc = tap - (tap / 3) * 3;
#pragma unroll
        for (int j = 0; j < NB; ++j)
          wf[bsel][j] = __builtin_bit_cast(bf16x8, wts[(RESW ? ck : 0) * C::W_CH + (tap * BN + cb0 + j * 32) * 4 + boff[kh]]);
#pragma unroll
        for (int m = 0; m < MB; ++m)
          hf[bsel][m] = __builtin_bit_cast(
              bf16x8, halo[aoff[UP ? dc : 0] + ((UP ? (m + dr + 1) >> 1 : m + dr) * SHW + (UP ? 0 : dc)) * C::HPITCH + 2 * kh]);
      };
      frag(0, 0);
#pragma unroll
      for (int i = 0; i < 18; ++i) {
        if (i + 1 < 18) frag(i + 1, (i + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);  // the reads stay ahead of this step's MFMAs
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[m][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i & 1][j], hf[i & 1][m], acc[m][j], 0, 0, 0);
      }
    }
    if (ticketed && !last && tid == 0) {
      s_next = 2 * n_x + static_cast<int>(ticket);
      // each workgroup draws one ticket too many; the last of those leaves
      // the counter at zero for the next launch
      if (ticket == static_cast<uint32_t>(band - n_x - 1))
        __hip_atomic_store(tickets + xcd * kTicketStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    epilogue(cur, false);  // with barriers between the write of s_next and its read
    if (last) break;
    cur = nxt;
    i_nxt = ticketed ? __builtin_amdgcn_readfirstlane(s_next) : band;
  }
}

// ------------------------------------------------------------- first layer
// The first conv (8 input channels, the last two zero) as a 72-deep
// contraction: two taps' 8 channels per 16-wide K slice, so a 32 x 32
// output block takes 5 v_mfma_f32_32x32x16_bf16 (the tenth tap slot has
// zero weights) where the general kernel takes 18 with K padded to 32.  One
// 8 x 32-pixel tile per workgroup; a halo pixel is one 16-byte LDS chunk
// (an odd pitch: fragment reads are free of bank conflicts), a weight row
// 11 chunks (10 tap slots and one of padding).
constexpr int kInTH = 8, kInHW = kTW + 2, kInHH = kInTH + 2, kInHalo = kInHH * kInHW, kInWP = 11;
// FRAME false reads the packed bf16 input x; true builds the input from a
// compositor frame's running mean and tile variance as it loads the halo
// (the values the frame glue writes: mean RGBA, log variance or 0 before two
// frames, 1/n, rounded to bf16 as the input packing does).
template <bool FRAME>
__global__ void __launch_bounds__(256) conv_in_k(Map x, FrameGlue fg,
                                                 const uint16_t* __restrict__ w, const float* __restrict__ bias, Map y,
                                                 Shape s) {
  constexpr int LDO = 40;  // staging row (one pixel) in bf16
  __shared__ __align__(16) uint4 halo[kInHalo];
  __shared__ __align__(16) uint4 wl[32 * kInWP];
  __shared__ __align__(16) uint16_t stg[kInTH * kTW * LDO];
  __shared__ __align__(16) float lb[32];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int tiles_x = (s.w + kTW - 1) / kTW, tiles_y = (s.h + kInTH - 1) / kInTH;
  const int t = static_cast<int>(blockIdx.x), n = t / (tiles_x * tiles_y), rr = t - n * tiles_x * tiles_y;
  const int oy0 = (rr / tiles_x) * kInTH, ox0 = (rr % tiles_x) * kTW;
  // halo pixels tid and tid + 256 (of kInHalo), image row oy0 - 1 + hr, column ox0 - 1 + hc
  uint4 hv[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = tid + 256 * k, hr = e / kInHW, hc = e - hr * kInHW, r = oy0 - 1 + hr, c = ox0 - 1 + hc;
    const int ok = (e < kInHalo) & (static_cast<unsigned>(r) < static_cast<unsigned>(s.h)) &
                   (static_cast<unsigned>(c) < static_cast<unsigned>(s.w));
    const int pix = r * s.w + c;  // within image n
    if (FRAME) {  // one image
      float4 mu = make_float4(0.f, 0.f, 0.f, 0.f);
      float lv = 0.f, inv_n = 0.f;
      if (ok) {
        const int ty = r / fg.tile_h, tx = c / fg.tile_w, t = ty * fg.tiles_x + tx;
        mu = reinterpret_cast<const float4*>(fg.accum)[static_cast<size_t>(t) * fg.P + (r - ty * fg.tile_h) * fg.tile_w +
                                                      (c - tx * fg.tile_w)];
        const float v = fg.tile_var[t];
        const int n_acc = fg.state->n_acc;
        lv = n_acc >= 2 ? logf(v > 1e-12f ? v : 1e-12f) : 0.f;
        inv_n = 1.f / static_cast<float>(n_acc);
      }
      hv[k] = uint4{pack_bf16(mu.x, mu.y), pack_bf16(mu.z, mu.w), pack_bf16(lv, inv_n), 0u};
    } else {
      const __amdgpu_buffer_rsrc_t src = buf_rsrc(x.p + x.off + static_cast<long long>(n) * s.h * s.w * x.ld);
      hv[k] = buf_load16(src, ok ? pix * x.ld * 2 : kOOB);
    }
  }
  // weights [tap][co][8] -> wl[co][tap] (tap slot 9 zero)
  const __amdgpu_buffer_rsrc_t wsrc = buf_rsrc(w);
  uint4 wv[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = tid + 256 * k, co = e / 10, tap = e - co * 10;
    wv[k] = buf_load16(wsrc, e < 320 && tap < 9 ? (tap * 32 + co) * 16 : kOOB);
  }
  if (tid < 32) lb[tid] = bias[tid];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = tid + 256 * k;
    if (e < kInHalo) halo[e] = hv[k];
    if (e < 320) wl[(e / 10) * kInWP + e % 10] = wv[k];
  }
  __syncthreads();
  // wave w: tile rows 2w, 2w + 1; slice i holds taps 2i (lanes 0-31) and 2i + 1 (lanes 32-63)
  f32x16 acc[2];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 b4 = *reinterpret_cast<const f32x4*>(lb + 8 * q + 4 * lh);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[m][4 * q + r] = b4[r];
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int tap = 2 * i + lh < 9 ? 2 * i + lh : 8, dr = tap / 3, dc = tap - (tap / 3) * 3;
    const bf16x8 a = __builtin_bit_cast(bf16x8, wl[l32 * kInWP + 2 * i + lh]);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const bf16x8 b = __builtin_bit_cast(bf16x8, halo[(2 * wave + m + dr) * kInHW + l32 + dc]);
      acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[m], 0, 0, 0);
    }
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<uint2*>(stg + ((2 * wave + m) * kTW + l32) * LDO + 8 * q + 4 * lh) =
          uint2{pack_bf16(fmaxf(acc[m][4 * q], 0.f), fmaxf(acc[m][4 * q + 1], 0.f)),
                pack_bf16(fmaxf(acc[m][4 * q + 2], 0.f), fmaxf(acc[m][4 * q + 3], 0.f))};
  __syncthreads();
  const __amdgpu_buffer_rsrc_t yb = buf_rsrc(y.p + y.off + ((static_cast<long long>(n) * s.h + oy0) * s.w + ox0) * y.ld);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int e = tid + 256 * k, px = e / 4, c = e % 4, row = px / kTW, col = px % kTW;
    const int ok = (oy0 + row < s.h) & (ox0 + col < s.w);
    buf_store16<kNT>(yb, ok ? ((row * s.w + col) * y.ld + c * 8) * 2 : kOOB,
                     *reinterpret_cast<const uint4*>(stg + px * LDO + c * 8));
  }
}

// ------------------------------------------------------- one-tile convolution
// conv3x3 with one TH x 32-pixel tile and 32 output channels per workgroup:
// the data gradients (dx[p] = sum over taps of W[tap]^T g[p - tap]), and the
// forward layers of maps with too few tiles for the persistent kernel to fill
// the chip.  4 waves, each MB tile rows (TH = 4 MB), in the persistent
// kernel's LDS layout.
//
// Forward: per 32-channel input slice the halo and the nine taps' weights are
// staged and the next slice is loaded into registers during the MFMAs, which
// take their operands in the persistent kernel's order (the same bits).
// Gradient: the halo of every slice is staged once and the weights follow in
// stages of TS taps, so that a sum runs over (tap, channel) in that order; with
// 32 output channels the two 16-channel halves of the slices are summed apart
// and added (two chains of MFMAs instead of one).
//
// The epilogue goes through an f32 staging tile, so that everything it reads
// and writes is 16 bytes of 8 channels with consecutive lanes on consecutive
// addresses, and does what were passes of their own over f32 maps: the ReLU
// gate of the layer below (g = bf16(dx * (y > 0))) with its bias gradient's
// partial sums, the adjoints of the 2x up-sampling and of the 2x2 pool (added
// to the skip's gradient).  Bound by latency: a workgroup's loads, MFMAs and
// epilogue are a few microseconds, so what counts is that a layer has
// workgroups for every compute unit and is one launch (8 x 128^2
// step: 27 launches of gates, gradients and adjoints 304 us, these 11 122).
enum TileEpi {
  kTileFwd = 0,   // y = bf16(relu(acc)), acc starting from the bias
  kTileFwdPool,   // ... and its 2x2 average
  kTileGate,      // g = bf16(acc * (y > 0)), channel groups from o.split on: skip = acc (f32)
  kTileUpGate,    // the same of the 2x2 sums (y, g at half the resolution)
  kTilePoolGate,  // g = bf16((skip + acc / 4) * (y > 0)) at twice the resolution
};

template <int NCH, int MB, bool UP, bool FWD>
struct TileCfg {
  static constexpr int TH = 4 * MB, SHH = UP ? TH / 2 + 2 : TH + 2, SHW = UP ? kTW / 2 + 2 : kTW + 2, HP = 5;
  static constexpr int HALO_CH = SHH * SHW * HP;                    // 16-byte chunks of a slice's halo
  static constexpr int TS = FWD || NCH == 1 ? 9 : NCH == 2 ? 3 : 1;  // taps of a weight stage
  static constexpr int WSL = FWD ? 1 : NCH;                         // input slices of a weight stage
  static constexpr int W_CH = TS * WSL * 32 * 4;
  static constexpr int WBUF = TS == 9 ? 1 : 2;
  static constexpr int PITCH = 36;  // staged floats of a pixel
  static constexpr int LOAD = (WSL * HALO_CH + WBUF * W_CH) * 16, STG = (TH * kTW * PITCH + 4 * 32) * 4;
  static constexpr int BYTES = LOAD > STG ? LOAD : STG;
};

template <int NCH, int MB, bool UP, int EPI, bool SPLIT>
__global__ void __launch_bounds__(256) conv_tile_k(Map x, Map x2, const uint16_t* __restrict__ w, int co_n,
                                                   const float* __restrict__ bias, TileOut o, Shape s) {
  constexpr bool FWD = EPI == kTileFwd || EPI == kTileFwdPool;
  using C = TileCfg<NCH, MB, UP, FWD>;
  static_assert(!(FWD && SPLIT) && !(UP && !FWD), "forward sums are one chain; gradients read no up-sampled map");
  constexpr int TH = C::TH, NT = 256, SHH = C::SHH, SHW = C::SHW, HP = C::HP, PITCH = C::PITCH;
  constexpr int HALO_EL = C::WSL * SHH * SHW * 4, W_CH = C::W_CH, CPP = C::WSL * 4;  // CPP: chunks loaded per pixel
  constexpr int HIT = (HALO_EL + NT - 1) / NT, WIT = (W_CH + NT - 1) / NT, CIN = NCH * 32;
  extern __shared__ __align__(16) uint4 lds4[];
  uint4* halo = lds4;                          // [WSL][SHH * SHW][HP]
  uint4* wts = lds4 + C::WSL * C::HALO_CH;     // [WBUF][TS][WSL][32][4]
  float* stg = reinterpret_cast<float*>(lds4);
  float* red = stg + TH * kTW * PITCH;         // [4][32]
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the channel groups of a tile, and the tiles of a band, on one XCD
  const int N = static_cast<int>(gridDim.x), xcd = static_cast<int>(blockIdx.x) % kXcds;
  const int id = xcd * (N / kXcds) + (xcd < N % kXcds ? xcd : N % kXcds) + static_cast<int>(blockIdx.x) / kXcds;
  const int groups = co_n / 32, tile = id / groups, grp = id - tile * groups, o0 = grp * 32;
  const int tiles_x = (s.w + kTW - 1) / kTW, tiles_y = (s.h + TH - 1) / TH;
  const int n = tile / (tiles_x * tiles_y), rem = tile - n * tiles_x * tiles_y;
  const int oy0 = (rem / tiles_x) * TH, ox0 = (rem % tiles_x) * kTW;
  const int hi = UP ? s.h / 2 : s.h, wi = UP ? s.w / 2 : s.w;  // the map x is read from
  const int sy0 = UP ? oy0 / 2 - 1 : oy0 - 1, sx0 = UP ? ox0 / 2 - 1 : ox0 - 1;

  int hoff[HIT];  // byte offset of this thread's halo chunks from the halo's top-left pixel
#pragma unroll
  for (int k = 0; k < HIT; ++k) {
    const int e = tid + NT * k, hp = e / CPP, cc = e % CPP, hr = hp / SHW, hc = hp - hr * SHW;
    const int ok = (e < HALO_EL) & (static_cast<unsigned>(sy0 + hr) < static_cast<unsigned>(hi)) &
                   (static_cast<unsigned>(sx0 + hc) < static_cast<unsigned>(wi));
    hoff[k] = ok ? ((hr * wi + hc) * x.ld + cc * 8) * 2 : kOOB;
  }
  const __amdgpu_buffer_rsrc_t wsrc = buf_rsrc(w);
  uint4 hreg[HIT], wreg[WIT];
  auto load_halo = [&](int ck) {
    const bool second = ck * kKC >= x.c;
    const Map& xm = second ? x2 : x;
    const int cb = second ? ck * kKC - x.c : ck * kKC;
    const __amdgpu_buffer_rsrc_t src =
        buf_rsrc(xm.p + xm.off + cb + (static_cast<long long>(n) * hi * wi + static_cast<long long>(sy0) * wi + sx0) * xm.ld);
#pragma unroll
    for (int k = 0; k < HIT; ++k) hreg[k] = buf_load16(src, hoff[k]);
  };
  auto load_w = [&](int tap0, int ck) {  // LDS row (tap, slice, channel)
#pragma unroll
    for (int k = 0; k < WIT; ++k) {
      const int e = tid + NT * k, row = e >> 2, co = row & 31, sl = (row >> 5) % C::WSL, tap = tap0 + (row >> 5) / C::WSL;
      wreg[k] = buf_load16(wsrc, e < W_CH ? ((tap * co_n + o0 + co) * CIN + (ck + sl) * kKC + (e & 3) * 8) * 2 : kOOB);
    }
  };
  auto store_halo = [&] {
#pragma unroll
    for (int k = 0; k < HIT; ++k) {
      const int e = tid + NT * k, cc = e % CPP;
      if (e < HALO_EL) halo[(cc >> 2) * C::HALO_CH + (e / CPP) * HP + (cc & 3)] = hreg[k];
    }
  };
  auto store_w = [&](int buf) {
#pragma unroll
    for (int k = 0; k < WIT; ++k) {
      const int e = tid + NT * k;
      if (e < W_CH) wts[buf * W_CH + swz(e >> 2, e & 3)] = wreg[k];
    }
  };
  load_halo(0);
  load_w(0, 0);
  f32x16 acc[MB][SPLIT ? 2 : 1];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f32x4 b4 = {0.f, 0.f, 0.f, 0.f};
    if constexpr (FWD) {  // the parameter vector's biases are 4-byte aligned
#pragma unroll
      for (int r = 0; r < 4; ++r) b4[r] = bias[o0 + 8 * q + 4 * lh + r];
    }
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int h = 0; h < (SPLIT ? 2 : 1); ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m][h][4 * q + r] = b4[r];
  }
  // fragment addresses as in the persistent kernel; halo row and column of
  // this lane's pixel in tile row m of the wave, moved by (dr, dc)
  const int boff[2] = {l32 * 4 + ((0 + lh) ^ ((l32 >> 2) & 3)), l32 * 4 + ((2 + lh) ^ ((l32 >> 2) & 3))};
  auto pixel = [&](int m, int dr, int dc) {
    const int row = wave * MB + m + dr;
    return UP ? ((row + 1) >> 1) * SHW + ((l32 + dc + 1) >> 1) : row * SHW + l32 + dc;
  };
  if constexpr (FWD) {
#pragma unroll
    for (int ck = 0; ck < NCH; ++ck) {
      if (ck) __syncthreads();  // the previous slice's fragment reads are done
      store_halo();
      store_w(0);
      __syncthreads();
      if (ck + 1 < NCH) {
        load_halo(ck + 1);
        load_w(0, ck + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
          const bf16x8 wf = __builtin_bit_cast(bf16x8, wts[tap * 32 * 4 + boff[kh]]);
#pragma unroll
          for (int m = 0; m < MB; ++m) {
            const bf16x8 hf = __builtin_bit_cast(bf16x8, halo[pixel(m, tap / 3, tap % 3) * HP + 2 * kh + lh]);
            acc[m][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, hf, acc[m][0], 0, 0, 0);
          }
        }
    }
  } else {
    store_halo();
#pragma unroll
    for (int st = 0; st < 9 / C::TS; ++st) {
      // into the buffer that stage st - 2 read: every wave is past it
      store_w(st % C::WBUF);
      __syncthreads();
      if (st + 1 < 9 / C::TS) load_w((st + 1) * C::TS, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < C::TS; ++t) {
        const int tap = st * C::TS + t, dr = 2 - tap / 3, dc = 2 - tap % 3;
#pragma unroll
        for (int sl = 0; sl < NCH; ++sl)
#pragma unroll
          for (int kh = 0; kh < 2; ++kh) {
            const bf16x8 wf =
                __builtin_bit_cast(bf16x8, wts[(st % C::WBUF) * W_CH + (t * NCH + sl) * 32 * 4 + boff[kh]]);
#pragma unroll
            for (int m = 0; m < MB; ++m) {
              const bf16x8 hf =
                  __builtin_bit_cast(bf16x8, halo[sl * C::HALO_CH + pixel(m, dr, dc) * HP + 2 * kh + lh]);
              f32x16& a = acc[m][SPLIT ? kh : 0];
              a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, hf, a, 0, 0, 0);
            }
          }
      }
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][0][r] += acc[m][1][r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x16& v = acc[m][0];
      *reinterpret_cast<f32x4*>(stg + ((wave * MB + m) * kTW + l32) * PITCH + 8 * q + 4 * lh) =
          f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    }
  __syncthreads();

  // items of 8 channels: chunk c8 of pixel px
  const int c8 = (tid & 3) * 8;
  auto staged = [&](int row, int col, float* v) {
    const f32x4* q = reinterpret_cast<const f32x4*>(stg + (row * kTW + col) * PITCH + c8);
    const f32x4 a = q[0], b = q[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = a[i];
      v[4 + i] = b[i];
    }
  };
  auto pack8 = [&](const float* v) {
    return uint4{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7])};
  };
  if constexpr (FWD) {
    uint16_t* yb = o.y.p + o.y.off + o0 + (static_cast<long long>(n) * s.h * s.w) * o.y.ld;
#pragma unroll
    for (int k = 0; k < TH * kTW / 64; ++k) {
      const int px = (tid >> 2) + 64 * k, r = oy0 + px / kTW, c = ox0 + px % kTW;
      float v[8];
      staged(px / kTW, px % kTW, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = fmaxf(v[i], 0.f);
      if (r < s.h && c < s.w) *reinterpret_cast<uint4*>(yb + (static_cast<long long>(r) * s.w + c) * o.y.ld + c8) = pack8(v);
    }
    if constexpr (EPI == kTileFwdPool) {
      const int ph = s.h / 2, pw = s.w / 2, q = tid >> 2;  // pooled pixel of the tile: ((a + b) + c) + d of the bf16 values
      uint16_t* pb = o.pool.p + o.pool.off + o0 + (static_cast<long long>(n) * ph * pw) * o.pool.ld;
      const int qr = q / (kTW / 2), qc = q % (kTW / 2), r = oy0 / 2 + qr, c = ox0 / 2 + qc;
      if (qr < TH / 2 && r < ph && c < pw) {
        float v[8], sum[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          staged(2 * qr + (k >> 1), 2 * qc + (k & 1), v);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float b = from_bf16(to_bf16(fmaxf(v[i], 0.f)));
            sum[i] = k ? sum[i] + b : b;
          }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) sum[i] *= 0.25f;
        *reinterpret_cast<uint4*>(pb + (static_cast<long long>(r) * pw + c) * o.pool.ld + c8) = pack8(sum);
      }
    }
    return;
  }
  if (EPI == kTileGate && grp >= o.split) {  // the skip half of a concatenation
    float* sb = o.skip + (static_cast<long long>(n) * s.h * s.w) * o.skip_ld + (grp - o.split) * 32 + c8;
#pragma unroll
    for (int k = 0; k < TH * kTW / 64; ++k) {
      const int px = (tid >> 2) + 64 * k, r = oy0 + px / kTW, c = ox0 + px % kTW;
      float v[8];
      staged(px / kTW, px % kTW, v);
      if (r < s.h && c < s.w) {
        f32x4* d = reinterpret_cast<f32x4*>(sb + (static_cast<long long>(r) * s.w + c) * o.skip_ld);
        d[0] = f32x4{v[0], v[1], v[2], v[3]};
        d[1] = f32x4{v[4], v[5], v[6], v[7]};
      }
    }
    return;
  }
  // the gated gradient of the layer below, at resolution gh x gw
  constexpr int ITEMS = EPI == kTileUpGate ? TH * kTW / 4 : EPI == kTilePoolGate ? TH * kTW * 4 : TH * kTW;  // pixels
  constexpr int GW = EPI == kTileUpGate ? kTW / 2 : EPI == kTilePoolGate ? kTW * 2 : kTW;                    // tile width
  const int gh = EPI == kTileUpGate ? s.h / 2 : EPI == kTilePoolGate ? s.h * 2 : s.h;
  const int gw = EPI == kTileUpGate ? s.w / 2 : EPI == kTilePoolGate ? s.w * 2 : s.w;
  const int gy0 = EPI == kTileUpGate ? oy0 / 2 : EPI == kTilePoolGate ? oy0 * 2 : oy0;
  const int gx0 = EPI == kTileUpGate ? ox0 / 2 : EPI == kTilePoolGate ? ox0 * 2 : ox0;
  const long long img = static_cast<long long>(n) * gh * gw;
  const uint16_t* yb = o.y.p + o.y.off + o0 + c8 + img * o.y.ld;
  uint16_t* gb = o.g.p + o.g.off + o0 + c8 + img * o.g.ld;
  const float* sb = o.skip + (EPI == kTilePoolGate ? img * o.skip_ld + o0 + c8 : 0);
  float sum[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) sum[i] = 0.f;
#pragma unroll 4
  for (int k = 0; k < (ITEMS + 63) / 64; ++k) {
    const int px = (tid >> 2) + 64 * k, pr = px / GW, pc = px % GW, r = gy0 + pr, c = gx0 + pc;
    if (px >= ITEMS || r >= gh || c >= gw) continue;
    const long long p = static_cast<long long>(r) * gw + c;
    const uint4 y4 = *reinterpret_cast<const uint4*>(yb + p * o.y.ld);
    float v[8];
    if constexpr (EPI == kTileUpGate) {
      staged(2 * pr, 2 * pc, v);
#pragma unroll
      for (int q = 1; q < 4; ++q) {
        float t[8];
        staged(2 * pr + (q >> 1), 2 * pc + (q & 1), t);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] += t[i];
      }
    } else if constexpr (EPI == kTilePoolGate) {
      const f32x4* sk = reinterpret_cast<const f32x4*>(sb + p * o.skip_ld);
      const f32x4 a = sk[0], b = sk[1];
      float t[8];
      staged(pr >> 1, pc >> 1, t);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = a[i] + 0.25f * t[i];
        v[4 + i] = b[i] + 0.25f * t[4 + i];
      }
    } else {
      staged(pr, pc, v);
    }
    const uint32_t yw[4] = {y4.x, y4.y, y4.z, y4.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float yi = (i & 1) ? bf16_hi(yw[i >> 1]) : bf16_lo(yw[i >> 1]);
      v[i] = yi > 0.f ? v[i] : 0.f;
      sum[i] += v[i];
    }
    *reinterpret_cast<uint4*>(gb + p * o.g.ld) = pack8(v);
  }
  // the tile's bias-gradient partial: over the 16 lanes of a chunk, then the waves
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    sum[i] += __shfl_xor(sum[i], 4, 64);
    sum[i] += __shfl_xor(sum[i], 8, 64);
    sum[i] += __shfl_xor(sum[i], 16, 64);
    sum[i] += __shfl_xor(sum[i], 32, 64);
  }
  if (lane < 4) {
#pragma unroll
    for (int i = 0; i < 8; ++i) red[wave * 32 + c8 + i] = sum[i];
  }
  __syncthreads();
  if (tid < 32)
    o.partial[static_cast<size_t>(tile) * o.g.c + o0 + tid] = ((red[tid] + red[32 + tid]) + red[64 + tid]) + red[96 + tid];
}

// ------------------------------------------------------------- wgrad
// dw[tap][ci][co] = sum_p x[p + tap][ci] g[p][co], g = bf16(dy * (y > 0)), of
// every conv layer in one launch.  A workgroup takes up to 64 x 64 (c_in,
// c_out) of one layer over a run of 8 x 32-pixel tiles; a wave holds one
// 32 x 32 block for all nine taps (144 accumulators), so a staged tile is
// read from memory once and not once per tap.  With fewer than four blocks
// the waves of a block split the tile's rows.
//
// x (with its halo) and g are staged as they lie in memory, [32-channel
// slice][pixel][32]; the operands need pixels along K, and
// ds_read_b64_tr_b16 transposes them on the way out: in each 16 lanes, lane
// 4 k + b addresses 4 channels of pixel k and lane l receives channel l of
// the 4 pixels (checked on the device).  A pixel's slice is 64 bytes, so the
// four pixels of 32 lanes cover the 64 banks once wherever they start, and a
// tap is an offset of whole pixels.  A row of x serves the three taps above,
// at and below it: three x operands and one g operand feed nine MFMAs.
//
// All layers in one launch because one layer's tiles fill the chip for only
// a few microseconds.  Bound by the latency of a tile's loads: its MFMAs take
// 0.5 to 2 us.  8 x 128^2 step, all 12 layers: 12 launches with one tap per
// workgroup 367 us, tiles staged through registers, x before g, 80 (with
// spills), straight into LDS 54.
constexpr int kWgTH = 8;                                // tile rows
constexpr int kWgXP = (kWgTH + 2) * (kTW + 2);          // halo pixels
constexpr int kWgGP = kWgTH * kTW;                      // pixels
constexpr int kWgAcc = 9 * 16;                          // accumulators of a wave
constexpr int kWgLds = 160 * 1024 / 2 / 16;             // 16-byte chunks of LDS: half a compute unit's
// s_waitcnt until at most n vector memory operations are outstanding (gfx9 encoding)
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
typedef short s16x4 __attribute__((ext_vector_type(4)));

// 16 pixels x 32 channels of a slice as an MFMA operand: this lane's channel,
// pixels 8 (lane / 32) .. + 7.  `at` is the lane's byte address of pixel 0.
__device__ __forceinline__ bf16x8 frag_tr(const char* at) {
  typedef __attribute__((address_space(3))) s16x4* P;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)(at));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)(at + 4 * 64));
  bf16x8 r;
  __builtin_memcpy(&r, &lo, 8);
  __builtin_memcpy(reinterpret_cast<char*>(&r) + 8, &hi, 8);
  return r;
}

// NR tile rows from the rows xr (halo) and gr point at.
template <int NR>
__device__ __forceinline__ void wgrad_rows(const char* xr, const char* gr, f32x16 (&acc)[9]) {
#pragma unroll
  for (int sg = 0; sg < kTW / 16; ++sg) {
    bf16x8 gv[3];
#pragma unroll
    for (int rr = 0; rr < NR + 2; ++rr) {
      bf16x8 xv[3];
#pragma unroll
      for (int dc = 0; dc < 3; ++dc) xv[dc] = frag_tr(xr + (rr * (kTW + 2) + sg * 16 + dc) * 64);
      if (rr < NR) gv[rr % 3] = frag_tr(gr + (rr * kTW + sg * 16) * 64);
#pragma unroll
      for (int dr = 0; dr < 3; ++dr) {
        if (rr - dr >= 0 && rr - dr < NR) {
#pragma unroll
          for (int dc = 0; dc < 3; ++dc)
            acc[dr * 3 + dc] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv[dc], gv[(rr - dr) % 3], acc[dr * 3 + dc], 0, 0, 0);
        }
      }
    }
  }
}

// 16 bytes from each lane's offset straight into LDS at `at` (wave-uniform) +
// 16 * lane; zeros where the offset is out of range.
__device__ __forceinline__ void buf_load_lds16(__amdgpu_buffer_rsrc_t r, uint4* at, int byte_off) {
  typedef __attribute__((address_space(3))) void* P;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (P)at, 16, byte_off, 0, 0, 0);
}

// One workgroup's share of layer L, a wave taking NR rows of a tile (8 / 4 / 2
// with 4 / 2 / 1 blocks), of CB c_in and OB c_out slices.  Tiles go straight
// from memory into LDS, x and g together, without passing through the
// registers the accumulators fill; the single blocks' tiles, whose MFMAs are
// the shortest, leave room for two and the next one is on its way meanwhile.
template <int CB, int OB>
__device__ __forceinline__ void wgrad_layer(const WgradLayer& L, int local, uint4* lds, float* __restrict__ partial) {
  constexpr int nblk = CB * OB, NR = 2 * nblk, rows = NR, parts = kWgTH / NR;
  constexpr int XIT = (CB * kWgXP * 4 + 255) / 256, GIT = OB * kWgGP * 4 / 256;
  constexpr int TILE_CH = (XIT + GIT) * 256, NBUF = nblk == 1 ? 2 : 1;  // 16-byte chunks of a staged tile
  static_assert(NBUF * TILE_CH <= kWgLds, "staged tiles fit");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ng = L.cig * L.cog, chunk = local / ng, group = local - chunk * ng;
  const int c0 = (group % L.cig) * CB * 32, o0 = (group / L.cig) * OB * 32;
  const int h = L.s.h, w = L.s.w, sw = L.up ? w / 2 : w, sh = L.up ? h / 2 : h, up = L.up;
  const int tiles_x = (w + kTW - 1) / kTW, tiles_y = (h + kWgTH - 1) / kWgTH, per_img = tiles_x * tiles_y;
  const int t0 = static_cast<int>(static_cast<long long>(chunk) * L.tiles / L.chunks);
  const int t1 = static_cast<int>(static_cast<long long>(chunk + 1) * L.tiles / L.chunks);
  // wave -> block (c_in slice, c_out slice) and part of the rows
  const int blk = wave % nblk, part = wave / nblk, bc = blk % CB, bo = blk / CB;
  const int l16 = lane & 15, lbyte = ((lane >> 5) * 8 + (l16 >> 2)) * 64 + ((lane >> 4) & 1) * 32 + (l16 & 3) * 8;
  const int r0 = part * rows;
  const int xat = (bc * kWgXP + r0 * (kTW + 2)) * 64 + lbyte, gat = XIT * 256 * 16 + (bo * kWgGP + r0 * kTW) * 64 + lbyte;
  f32x16 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
  // this thread's chunk k of x: slice, halo pixel (row, column) and 8 channels
  // (one past the last is padding: no channel), packed as row | column << 8 |
  // channel << 16, kept while the accumulators take the other registers
  const int xld = L.xld, co = L.co;
  const long long ximg = static_cast<long long>(sh) * sw * xld, gimg = static_cast<long long>(h) * w * co;
  const uint16_t *xp = L.x, *gp = L.g;
  int xe[XIT];
#pragma unroll
  for (int k = 0; k < XIT; ++k) {
    const int e = tid + 256 * k, sl = e / (kWgXP * 4), q = e - sl * (kWgXP * 4), px = q >> 2, hr = px / (kTW + 2);
    const int ch = c0 + sl * 32 + (q & 3) * 8;
    xe[k] = sl < CB && ch < L.xc ? hr | (px - hr * (kTW + 2)) << 8 | ch << 16 : 0xFF;  // row 255 is outside every tile
  }
  auto stage = [&](int t, uint4* to) {
    const int n = t / per_img, rem = t - n * per_img, oy = (rem / tiles_x) * kWgTH, ox = (rem % tiles_x) * kTW;
    const __amdgpu_buffer_rsrc_t xb = buf_rsrc(xp + n * ximg), gb = buf_rsrc(gp + n * gimg);
    uint4* at = to + wave * 64;
#pragma unroll
    for (int k = 0; k < XIT; ++k) {
      const int hr = xe[k] & 0xFF, r = oy - 1 + hr, c = ox - 1 + ((xe[k] >> 8) & 0xFF);
      int off = ((up ? (r >> 1) * sw + (c >> 1) : r * sw + c) * xld + (xe[k] >> 16)) * 2;
      asm("" : "+v"(off));  // selected, not branched around
      const bool ok = (hr < kWgTH + 2) & (static_cast<unsigned>(r) < static_cast<unsigned>(h)) &
                      (static_cast<unsigned>(c) < static_cast<unsigned>(w));
      buf_load_lds16(xb, at + 256 * k, ok ? off : kOOB);
    }
    const int gr = oy + (tid >> 7), gc = ox + ((tid >> 2) & 31);  // chunk k: two rows on from chunk k - 1
    int goff = ((gr * w + gc) * co + o0 + (tid & 3) * 8) * 2;
    asm("" : "+v"(goff));
#pragma unroll
    for (int k = 0; k < GIT; ++k) {
      const int sl = k / 4, row = 2 * (k % 4);
      const bool ok = (gr + row < h) & (gc < w);
      buf_load_lds16(gb, at + 256 * (XIT + k), ok ? goff + (row * w * co + sl * 32) * 2 : kOOB);
    }
  };
  int buf = 0;
  if (NBUF == 2 && t0 < t1) stage(t0, lds);
  for (int t = t0; t < t1; ++t) {
    if (NBUF == 2) {
      if (t + 1 < t1) {
        stage(t + 1, lds + (buf ^ 1) * TILE_CH);
        __builtin_amdgcn_s_waitcnt(wait_vm(XIT + GIT));  // the tile before it has arrived
      } else {
        __builtin_amdgcn_s_waitcnt(wait_vm(0));
      }
    } else {
      stage(t, lds);
      __builtin_amdgcn_s_waitcnt(wait_vm(0));
    }
    lds_barrier();
    const char* tile = reinterpret_cast<const char*>(lds + buf * TILE_CH);
    wgrad_rows<NR>(tile + xat, tile + gat, acc);
    lds_barrier();  // every wave is done with the tile
    if (NBUF == 2) buf ^= 1;
  }
  // the parts of a block, added in a fixed order: 2 and 3 to 0 and 1, then 1 to 0
  float* red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int half = parts / 2; half > 0; half /= 2) {
    __syncthreads();
    if (part >= half && part < 2 * half) {
      float* q = red + ((part - half) * nblk + blk) * kWgAcc * 64 + lane;
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) q[(t * 16 + r) * 64] = acc[t][r];
    }
    __syncthreads();
    if (part < half) {
      const float* q = red + (part * nblk + blk) * kWgAcc * 64 + lane;
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] += q[(t * 16 + r) * 64];
    }
  }
  if (part == 0) {
    float* q = partial + L.part + (static_cast<size_t>(local) * nblk + blk) * kWgAcc * 64 + lane;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) q[(t * 16 + r) * 64] = acc[t][r];
  }
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
wgrad_k(WgradPlan plan, float* __restrict__ partial) {
  __shared__ __align__(16) uint4 lds[kWgLds];
  const int bid = static_cast<int>(blockIdx.x);
  int li = 0;
  for (int i = 1; i < kConvLayers; ++i)
    if (bid >= plan.l[i].first_wg) li = i;
  const WgradLayer& L = plan.l[li];
  if (L.cb == 2 && L.ob == 2) wgrad_layer<2, 2>(L, bid - L.first_wg, lds, partial);
  else if (L.cb == 2) wgrad_layer<2, 1>(L, bid - L.first_wg, lds, partial);
  else if (L.ob == 2) wgrad_layer<1, 2>(L, bid - L.first_wg, lds, partial);
  else wgrad_layer<1, 1>(L, bid - L.first_wg, lds, partial);
}

// ------------------------------------------------------- gradient sums, Adam
__device__ __forceinline__ float adam_step(float w, float gi, float& m, float& v, const AdamArgs& a) {
  const float mi = a.b1 * m + (1.f - a.b1) * gi;
  const float vi = a.b2 * v + (1.f - a.b2) * gi * gi;
  m = mi;
  v = vi;
  return w - a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
}

// Every parameter's gradient from its partial sums (added in a fixed order)
// and, with a.update, its Adam step and its bf16 copies, in one launch (38
// launches before: two sums a layer, Adam, a copy a layer; 8 x 128^2 step:
// 199 us, now 23).  The first plan.conv_blocks workgroups take 256 conv weights each, in the order
// the weight gradient's accumulators were stored; the others one bias, output
// conv parameter or the loss sum each.
__global__ void __launch_bounds__(256) update_k(UpdatePlan plan, const float* __restrict__ partial, AdamArgs a) {
  __shared__ float red[256];
  const int t = threadIdx.x, bid = static_cast<int>(blockIdx.x);
  if (bid < plan.conv_blocks) {
    int li = 0;
    for (int i = 1; i < kConvLayers; ++i)
      if (bid >= plan.l[i].first_block) li = i;
    const UpdateLayer& L = plan.l[li];
    const int e = (bid - L.first_block) * 256 + t;  // [group][block][tap][r][lane]
    const int nblk = L.cb * L.ob, gb = e / (kWgAcc * 64), q = e - gb * (kWgAcc * 64), group = gb / nblk, blk = gb - group * nblk;
    const int tap = q >> 10, r = (q >> 6) & 15, lane = q & 63;
    const int ci = ((group % L.cig) * L.cb + blk % L.cb) * 32 + 8 * (r / 4) + 4 * (lane >> 5) + r % 4;
    const int co = ((group / L.cig) * L.ob + blk / L.cb) * 32 + (lane & 31);
    if (ci >= L.ci) return;
    const size_t step = static_cast<size_t>(L.cig * L.cog) * nblk * kWgAcc * 64;
    const float* p = partial + L.part + e;
    float s4[4] = {0.f, 0.f, 0.f, 0.f};
    int c = 0;
    for (; c + 4 <= L.chunks; c += 4)
#pragma unroll
      for (int k = 0; k < 4; ++k) s4[k] += p[(c + k) * step];
    for (; c < L.chunks; ++c) s4[0] += p[c * step];
    const float gi = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    const int i = L.off_w + (tap * L.ci + ci) * L.co + co;
    a.g[i] = gi;
    if (a.update) {
      const float wn = adam_step(a.w[i], gi, a.m[i], a.v[i], a);
      a.w[i] = wn;
      const uint16_t hb = to_bf16(wn);
      L.wd[(tap * L.ci_pad + ci) * L.co + co] = hb;
      L.wf[(tap * L.co + co) * L.ci_pad + ci] = hb;
    }
    return;
  }
  int o = bid - plan.conv_blocks, li = 0;
  for (int i = 1; i <= kConvLayers; ++i)
    if (o >= plan.bias[i].first) li = i;
  const BiasPart& B = plan.bias[li];
  o -= B.first;
  const float* p = partial + B.part + o;
  float sum = 0.f;
  for (int c = t; c < B.rows; c += 256) sum += p[static_cast<size_t>(c) * B.n];
  red[t] = sum;
  __syncthreads();
  for (int hf = 128; hf > 0; hf >>= 1) {
    if (t < hf) red[t] += red[t + hf];
    __syncthreads();
  }
  if (t == 0) {
    const float gi = red[0];
    if (li == kConvLayers && o == B.n - 1) {  // the output conv's last column is the loss
      *a.loss = gi;
    } else {
      const int i = B.param + o;
      a.g[i] = gi;
      if (a.update) a.w[i] = adam_step(a.w[i], gi, a.m[i], a.v[i], a);
    }
  }
}

// ------------------------------------------------------------- glue kernels
__global__ void out_fwd_k(Map x, const float* __restrict__ w, const float* __restrict__ b,
                          const float* __restrict__ base, int base_ld, float* __restrict__ out, Shape s) {
  const long long p = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= s.pixels()) return;
  float o0 = base[p * base_ld] + b[0], o1 = base[p * base_ld + 1] + b[1], o2 = base[p * base_ld + 2] + b[2];
  float a0 = 0.f, a1 = 0.f, a2 = 0.f;
  const uint16_t* row = x.p + p * x.ld + x.off;
  for (int i0 = 0; i0 < x.c; i0 += 8) {  // x.c, ld and off are multiples of 8
    const uint4 v = *reinterpret_cast<const uint4*>(row + i0);
    const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = i0 + k;
      const float xi = from_bf16(static_cast<uint16_t>(vw[k >> 1] >> ((k & 1) * 16)));
      a0 = fmaf(xi, w[i * 3 + 0], a0);
      a1 = fmaf(xi, w[i * 3 + 1], a1);
      a2 = fmaf(xi, w[i * 3 + 2], a2);
    }
  }
  out[p * 3 + 0] = o0 + a0;
  out[p * 3 + 1] = o1 + a1;
  out[p * 3 + 2] = o2 + a2;
}

// The output conv, the loss and their gradients in one pass over the last
// layer's output x (bf16, 32 channels): out = base + b + x w, dout = 2 (out -
// t) / count, dx = dout w^T, g = bf16(dx * (x > 0)), the gated gradient of the
// last conv layer.  Per chunk of kOutChunk pixels: bias[chunk][32] = sum g in
// f32, and partial[chunk] = {dw[ci][3], db[3], sum (out - t)^2}.  Four lanes
// share a pixel, 8 channels each; a lane's sums over its pixels are added over
// the lanes and waves in a fixed order.  (Three passes with an f32 dx and 2
// bytes a lane took 31 us
// of the 8 x 128^2 step, this 13.)
constexpr int kOutChunk = 256;
__global__ void __launch_bounds__(256) out_bwd_k(Map x, const float* __restrict__ base, int base_ld,
                                                 const float* __restrict__ tgt, const float* __restrict__ w,
                                                 const float* __restrict__ b, Map g, float* __restrict__ bias,
                                                 float* __restrict__ partial, long long P, float scale) {
  __shared__ float red[4][36 * 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = tid & 3;
  float wl[8][3];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) wl[i][c] = w[(q * 8 + i) * 3 + c];
  // 24 dw, 8 sums of g, 3 db and the loss (the last four the same in all lanes of a pixel)
  float v[36];
#pragma unroll
  for (int i = 0; i < 36; ++i) v[i] = 0.f;
  const long long p0 = static_cast<long long>(blockIdx.x) * kOutChunk;
#pragma unroll
  for (int k = 0; k < kOutChunk / 64; ++k) {
    const long long p = p0 + (tid >> 2) + 64 * k;
    const bool ok = p < P;
    // every lane takes the whole row, so that the sums run in channel order
    float a[3] = {0.f, 0.f, 0.f}, xi[8], d[3];
#pragma unroll
    for (int i = 0; i < 8; ++i) xi[i] = 0.f;
#pragma unroll
    for (int c8 = 0; c8 < 4; ++c8) {
      uint4 x4 = {0u, 0u, 0u, 0u};
      if (ok) x4 = *reinterpret_cast<const uint4*>(x.p + p * x.ld + x.off + c8 * 8);
      const uint32_t xw[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float f = (i & 1) ? bf16_hi(xw[i >> 1]) : bf16_lo(xw[i >> 1]);
        if (c8 == q) xi[i] = f;
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = fmaf(f, w[(c8 * 8 + i) * 3 + c], a[c]);
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float e = ok ? ((base[p * base_ld + c] + b[c]) + a[c]) - tgt[p * 3 + c] : 0.f;
      d[c] = scale * e;
      v[32 + c] += d[c];
      v[35] = fmaf(e, e, v[35]);
    }
    float gi[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int c = 0; c < 3; ++c) v[i * 3 + c] = fmaf(xi[i], d[c], v[i * 3 + c]);
      gi[i] = xi[i] > 0.f ? d[0] * wl[i][0] + d[1] * wl[i][1] + d[2] * wl[i][2] : 0.f;
      v[24 + i] += gi[i];
    }
    if (ok)
      *reinterpret_cast<uint4*>(g.p + p * g.ld + g.off + q * 8) =
          uint4{pack_bf16(gi[0], gi[1]), pack_bf16(gi[2], gi[3]), pack_bf16(gi[4], gi[5]), pack_bf16(gi[6], gi[7])};
  }
#pragma unroll
  for (int i = 0; i < 36; ++i) {
    v[i] += __shfl_xor(v[i], 4, 64);
    v[i] += __shfl_xor(v[i], 8, 64);
    v[i] += __shfl_xor(v[i], 16, 64);
    v[i] += __shfl_xor(v[i], 32, 64);
  }
  if (lane < 4) {
#pragma unroll
    for (int i = 0; i < 36; ++i) red[wave][q * 36 + i] = v[i];
  }
  __syncthreads();
  if (tid < 36 * 4) {
    const float sum = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
    const int qq = tid / 36, i = tid - qq * 36;
    float* out = partial + static_cast<size_t>(blockIdx.x) * 100;
    if (i < 24) out[qq * 24 + i] = sum;
    else if (i < 32) bias[static_cast<size_t>(blockIdx.x) * 32 + qq * 8 + i - 24] = sum;
    else if (qq == 0) out[96 + i - 32] = sum;
  }
}

// one thread per pixel: 6 f32 in, one 16-byte store of 8 bf16 (channels 6, 7 zero)
__global__ void pack_input_k(const float* __restrict__ in, int in_ld, uint16_t* __restrict__ x, long long P) {
  const long long p = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= P) return;
  const float* q = in + p * in_ld;
  uint32_t h[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) h[c] = to_bf16(q[c]);
  *reinterpret_cast<uint4*>(x + p * 8) = uint4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), 0u};
}

// master [9][ci][co] -> fwd [9][co][ci_pad] and dgrad [9][ci_pad][co] (bf16,
// channels ci..ci_pad-1 zero)
__global__ void refresh_k(const float* __restrict__ wm, uint16_t* __restrict__ wf, uint16_t* __restrict__ wd,
                          int ci, int ci_pad, int co) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 9 * ci_pad * co) return;
  const int o = e % co, i = (e / co) % ci_pad, t = e / (co * ci_pad);
  const uint16_t h = i < ci ? to_bf16(wm[(static_cast<size_t>(t) * ci + i) * co + o]) : static_cast<uint16_t>(0);
  wd[(static_cast<size_t>(t) * ci_pad + i) * co + o] = h;
  wf[(static_cast<size_t>(t) * co + o) * ci_pad + i] = h;
}

// ------------------------------------------------------------- frame glue
__global__ void frame_to_input_k(FrameGlue g, float* __restrict__ in6) {
  const long long p = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  const long long P = static_cast<long long>(g.width) * g.height;
  if (p >= P) return;
  const int y = static_cast<int>(p / g.width), x = static_cast<int>(p - static_cast<long long>(y) * g.width);
  const int t = (y / g.tile_h) * g.tiles_x + x / g.tile_w;
  const int q = (y % g.tile_h) * g.tile_w + x % g.tile_w;
  const float4 mu = reinterpret_cast<const float4*>(g.accum)[static_cast<size_t>(t) * g.P + q];
  const float v = g.tile_var[t];
  float* o = in6 + p * 6;
  o[0] = mu.x;
  o[1] = mu.y;
  o[2] = mu.z;
  o[3] = mu.w;
  const int n_acc = g.state->n_acc;
  o[4] = n_acc >= 2 ? logf(v > 1e-12f ? v : 1e-12f) : 0.f;
  o[5] = 1.f / static_cast<float>(n_acc);
}

// display quantisation of one channel to 8 bits (optional gamma)
__device__ __forceinline__ uint32_t q8(float x, bool gamma, float inv_gamma) {
  float y = x > 0.f ? x : 0.f;
  y = y < 1.f ? y : 1.f;
  if (gamma) y = powf(y, inv_gamma);
  return static_cast<uint32_t>(floorf(fmaf(255.f, y, 0.5f)));
}

// The frame's display buffer from its denoised pixels; the padding pixels of
// ragged edge tiles, which the network does not see, take the running mean
// (in den too).
__global__ void frame_display_k(FrameGlue g, float* __restrict__ den, void* final_out, uint32_t mode,
                                float inv_gamma) {
  const long long e = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int T = g.tiles_x * ((g.height + g.tile_h - 1) / g.tile_h);
  if (e >= static_cast<long long>(T) * g.P) return;
  const int t = static_cast<int>(e / g.P), q = static_cast<int>(e - static_cast<long long>(t) * g.P);
  const int x = (t % g.tiles_x) * g.tile_w + q % g.tile_w;
  const int y = (t / g.tiles_x) * g.tile_h + q / g.tile_w;
  float4 v;
  if (x < g.width && y < g.height) {
    v = reinterpret_cast<const float4*>(den)[e];
  } else {
    v = reinterpret_cast<const float4*>(g.accum)[e];
    reinterpret_cast<float4*>(den)[e] = v;
  }
  if (mode & kModeFmtRGBA8) {
    const bool gm = (mode & kModeGamma) != 0;
    static_cast<uint32_t*>(final_out)[e] = q8(v.x, gm, inv_gamma) | (q8(v.y, gm, inv_gamma) << 8) |
                                           (q8(v.z, gm, inv_gamma) << 16) | (q8(v.w, false, 1.f) << 24);
  } else if (mode & kModeFmtF32) {
    static_cast<float4*>(final_out)[e] = v;
  }
}

inline unsigned blocks(long long n, int t) { return static_cast<unsigned>((n + t - 1) / t); }

}  // namespace

template <int BN, int CP, int TH, bool UP, int EPI>
hipError_t launch_conv(const Map& x, const Map& x2, const uint16_t* w, const float* bias, const Map& y, const Map& pool,
                       const OutConv& oc, const Shape& s, uint32_t* tickets, hipStream_t st) {
  using C = ConvCfg<BN, TH, CP / kKC, UP>;
  const void* f = reinterpret_cast<const void*>(&conv_fwd_k<BN, CP, TH, UP, EPI>);
  const size_t lds = C::BYTES + (EPI == kEpiFrame ? 99 * 4 : 0);
  const long long tiles = static_cast<long long>(s.n) * ((s.h + TH - 1) / TH) * ((s.w + kTW - 1) / kTW);
  if (tiles == 0) return hipSuccess;
  if (tiles > (1LL << 30)) return hipErrorInvalidValue;
  // resident workgroups per compute unit, per device
  static int per_cu[64] = {0};
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (lds > 64 * 1024) {
    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  if (per_cu[dev] == 0) {
    int nb = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, C::NT, lds);
    if (e != hipSuccess) return e;
    per_cu[dev] = nb > 0 ? nb : 1;
  }
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const long long grid = tiles < static_cast<long long>(cus) * per_cu[dev] ? tiles : static_cast<long long>(cus) * per_cu[dev];
  conv_fwd_k<BN, CP, TH, UP, EPI><<<static_cast<unsigned>(grid), C::NT, lds, st>>>(x, x2, w, bias, y, pool, oc, s, tickets);
  return hipGetLastError();
}

template <int BN, int CP, int TH, bool UP>
hipError_t launch_tile(const Map& x, const Map& x2, const uint16_t* w, const float* bias, const Map& y,
                       const Map& pool, const Shape& s, uint32_t* tickets, hipStream_t st) {
  const OutConv none{nullptr, nullptr, FrameGlue{}, 0.f, nullptr};
  if (pool.p) {
    if constexpr ((TH / 4) % 2 == 0) return launch_conv<BN, CP, TH, UP, kEpiPool>(x, x2, w, bias, y, pool, none, s, tickets, st);
    return hipErrorInvalidValue;
  }
  return launch_conv<BN, CP, TH, UP, kEpiPlain>(x, x2, w, bias, y, pool, none, s, tickets, st);
}

// Rows of a one-tile convolution's tiles: 8, or 4 where 8 leave fewer than two
// workgroups for each of 256 compute units (8 x 128^2
// step, all kernels: from 256 workgroups on 384 us, from 512 379, from 1024
// 387).
#ifndef DFB_TILE_MIN
#define DFB_TILE_MIN 512
#endif
constexpr int kTileMin = DFB_TILE_MIN;
int tile_rows(const Shape& s, int co) {
  const long long tiles = static_cast<long long>(s.n) * ((s.h + 7) / 8) * ((s.w + kTW - 1) / kTW);
  return tiles * (co / 32) >= kTileMin ? 8 : 4;
}
int conv_tiles(const Shape& s, int co) {
  const int th = tile_rows(s, co);
  return static_cast<int>(static_cast<long long>(s.n) * ((s.h + th - 1) / th) * ((s.w + kTW - 1) / kTW));
}

template <int NCH, int MB, bool UP, int EPI, bool SPLIT>
hipError_t launch_tile_conv(const Map& x, const Map& x2, const uint16_t* w, int co, const float* bias, const TileOut& o,
                            const Shape& s, hipStream_t st) {
  using C = TileCfg<NCH, MB, UP, EPI == kTileFwd || EPI == kTileFwdPool>;
  if (C::BYTES > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_tile_k<NCH, MB, UP, EPI, SPLIT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, C::BYTES);
    if (e != hipSuccess) return e;
  }
  conv_tile_k<NCH, MB, UP, EPI, SPLIT>
      <<<static_cast<unsigned>(conv_tiles(s, co) * (co / 32)), 256, C::BYTES, st>>>(x, x2, w, co, bias, o, s);
  return hipGetLastError();
}
// Output tiles from which a forward layer takes the persistent kernel: with
// fewer, some of 256 compute units are left without a workgroup, and the one-tile kernel's
// 32-channel groups and 4-row tiles fill them (8 x 128^2 training: the seven
// layers below it 104 -> 56 us; with 256 to 512 tiles the two are within a
// microsecond).
#ifndef DFB_PERSIST_MIN
#define DFB_PERSIST_MIN 256
#endif
constexpr int kPersistMin = DFB_PERSIST_MIN;
template <bool UP, int CIN>
hipError_t tile_fwd(const Map& x, const Map& x2, const uint16_t* w, const float* bias, const Map& y, const Map& pool,
                    const Shape& s, hipStream_t st) {
  const Map none{nullptr, 0, 0, 0};
  const TileOut o{y, none, pool, nullptr, 0, 0, nullptr};
  const bool tall = tile_rows(s, y.c) == 8;
#define DFB_TILE(EPI_)                                                                                   \
  return tall ? launch_tile_conv<CIN / 32, 2, UP, EPI_, false>(x, x2, w, y.c, bias, o, s, st)              \
              : launch_tile_conv<CIN / 32, 1, UP, EPI_, false>(x, x2, w, y.c, bias, o, s, st)
  if (pool.p) DFB_TILE(kTileFwdPool);
  DFB_TILE(kTileFwd);
#undef DFB_TILE
}

template <bool UP>
hipError_t conv_tile(const Map& x, const Map& x2, const uint16_t* w, const float* bias, const Map& y,
                     const Map& pool, const Shape& s, uint32_t* tickets, hipStream_t st) {
  const int cp = (x.c + x2.c + 31) / 32 * 32;
#define DFB_CONV(BN_, CP_, TH_, THU_)                                                                               \
  if (y.c == BN_ && cp == CP_) {                                                                                    \
    constexpr int TH = UP ? THU_ : TH_;                                                                             \
    if (cp == x.c + x2.c && static_cast<long long>(s.n) * ((s.h + TH - 1) / TH) * ((s.w + kTW - 1) / kTW) < kPersistMin) \
      return tile_fwd<UP, CP_>(x, x2, w, bias, y, pool, s, st);                                                     \
    return launch_tile<BN_, CP_, TH, UP>(x, x2, w, bias, y, pool, s, tickets, st);                                  \
  }
  DFB_CONV(32, 32, DFB_TH_32_32, DFB_TH_32_32)
  DFB_CONV(32, 64, DFB_TH_32_64, DFB_THU_32_64)
  DFB_CONV(64, 32, DFB_TH_64_32, DFB_TH_64_32)
  DFB_CONV(64, 64, DFB_TH_64_64, DFB_TH_64_64)
  DFB_CONV(64, 128, DFB_TH_64_128, DFB_THU_64_128)
  DFB_CONV(128, 64, DFB_TH_128, DFB_TH_128)
  DFB_CONV(128, 128, DFB_TH_128, DFB_TH_128)
#undef DFB_CONV
  return hipErrorInvalidValue;
}

hipError_t conv3x3_fwd(const Map& x, const uint16_t* w_fwd, const float* bias, const Map& y, const Shape& s,
                       uint32_t* tickets, hipStream_t st, bool up, const Map* pool, const Map* x2) {
  const Map none{nullptr, 0, 0, 0};
  const Map& xb = x2 ? *x2 : none;
  if (x.c % 8 || x.ld % 8 || x.off % 8 || y.ld % 8 || y.off % 8) return hipErrorInvalidValue;
  if (x2 && (x.c % 32 || xb.c % 8 || xb.ld != x.ld || xb.off % 8)) return hipErrorInvalidValue;
  if ((up || pool) && (s.h % 2 || s.w % 2)) return hipErrorInvalidValue;
  // per-image element offsets are 32-bit
  const long long img = static_cast<long long>(up ? s.h / 2 : s.h) * (up ? s.w / 2 : s.w) * x.ld;
  if (img >= (1LL << 30) || static_cast<long long>(s.h) * s.w * y.ld >= (1LL << 30)) return hipErrorInvalidValue;
  const Map& pl = pool ? *pool : none;
  if (pool && (pl.ld % 8 || pl.off % 8 || pl.c != y.c)) return hipErrorInvalidValue;
  return up ? conv_tile<true>(x, xb, w_fwd, bias, y, pl, s, tickets, st)
            : conv_tile<false>(x, xb, w_fwd, bias, y, pl, s, tickets, st);
}

// The data gradient from `in` channels to ci.
template <int EPI>
hipError_t tile_bwd(const Map& g, const uint16_t* w, int ci, const TileOut& o, const Shape& s, hipStream_t st) {
  const Map none{nullptr, 0, 0, 0};
  const bool tall = tile_rows(s, ci) == 8;
#define DFB_TILE(C_, MB_, SPLIT_) return launch_tile_conv<C_ / 32, MB_, false, EPI, SPLIT_>(g, none, w, ci, nullptr, o, s, st)
#define DFB_TILES(C_)                                    \
  case C_:                                               \
    if (ci == 32 && tall) DFB_TILE(C_, 2, true);         \
    if (ci == 32) DFB_TILE(C_, 1, true);                 \
    if (tall) DFB_TILE(C_, 2, false);                    \
    DFB_TILE(C_, 1, false);
  switch (g.c) {
    DFB_TILES(32)
    DFB_TILES(64)
    DFB_TILES(128)
  }
#undef DFB_TILES
#undef DFB_TILE
  return hipErrorInvalidValue;
}

hipError_t conv3x3_bwd(const Map& g, const uint16_t* w_dgrad, int ci, Adjoint adj, const TileOut& o, const Shape& s,
                       hipStream_t st) {
  if (g.ld % 8 || g.off % 8 || o.y.ld % 8 || o.y.off % 8 || o.g.ld % 8 || o.g.off % 8 || o.skip_ld % 4 || ci % 32)
    return hipErrorInvalidValue;
  // per-image byte offsets of g are 32-bit
  if (static_cast<long long>(s.h) * s.w * g.ld >= (1LL << 30)) return hipErrorInvalidValue;
  if (conv_tiles(s, ci) == 0) return hipSuccess;
  switch (adj) {
    case Adjoint::kSame: return tile_bwd<kTileGate>(g, w_dgrad, ci, o, s, st);
    case Adjoint::kUp: return tile_bwd<kTileUpGate>(g, w_dgrad, ci, o, s, st);
    case Adjoint::kPool: return tile_bwd<kTilePoolGate>(g, w_dgrad, ci, o, s, st);
  }
  return hipErrorInvalidValue;
}

// Workgroups of the weight-gradient launch at most, per layer (rows of 64 x 64
// channel groups included): the layers' shares of about 512, two for each of
// 256 compute units, by their tiles at the three resolutions and the cycles of a
// tile (its MFMAs, and as much again to stage it for the 32-channel layers).
int wgrad_chunks(int layer, long long tiles) {
  static const int cap[kConvLayers] = {51, 51, 17, 27, 7, 7, 27, 27, 27, 70, 70, 51};
  return static_cast<int>(tiles < cap[layer] ? (tiles < 1 ? 1 : tiles) : cap[layer]);
}
long long wgrad_tiles(const Shape& s) {
  return static_cast<long long>(s.n) * ((s.h + kWgTH - 1) / kWgTH) * ((s.w + kTW - 1) / kTW);
}
size_t wgrad_floats(const WgradLayer& L) {
  return static_cast<size_t>(L.chunks) * L.cig * L.cog * L.cb * L.ob * kWgAcc * 64;
}

hipError_t conv3x3_wgrad(const WgradPlan& plan, float* partial, hipStream_t st) {
  for (const WgradLayer& L : plan.l) {
    if (L.xld % 8 || L.xc % 8 || L.co % 32 || reinterpret_cast<uintptr_t>(L.x) % 16 || reinterpret_cast<uintptr_t>(L.g) % 16)
      return hipErrorInvalidValue;
    const long long img = static_cast<long long>(L.s.h) * L.s.w;  // per-image byte offsets are 32-bit
    if (img * L.xld >= (1LL << 30) || img * L.co >= (1LL << 30)) return hipErrorInvalidValue;
  }
  wgrad_k<<<static_cast<unsigned>(plan.n_wg), 256, 0, st>>>(plan, partial);
  return hipGetLastError();
}

int update_blocks(const UpdateLayer& L) { return L.cig * L.cog * L.cb * L.ob * kWgAcc * 64 / 256; }

hipError_t update_params(const UpdatePlan& plan, const float* partial, const AdamArgs& a, hipStream_t st) {
  const int n = plan.conv_blocks + plan.bias[kConvLayers].first + plan.bias[kConvLayers].n;
  update_k<<<static_cast<unsigned>(n), 256, 0, st>>>(plan, partial, a);
  return hipGetLastError();
}

hipError_t conv3x3_in_fwd(const Map& x, const uint16_t* w_fwd, const float* bias, const Map& y, const Shape& s,
                          hipStream_t st) {
  if (y.c != 32 || y.ld % 8 || y.off % 8) return hipErrorInvalidValue;
  if (x.c != 8 || x.ld % 8 || x.off % 8) return hipErrorInvalidValue;
  const long long img = static_cast<long long>(s.h) * s.w;
  if (img * x.ld * 2 >= (1LL << 31) || img * y.ld >= (1LL << 30)) return hipErrorInvalidValue;
  const long long tiles = static_cast<long long>(s.n) * ((s.h + kInTH - 1) / kInTH) * ((s.w + kTW - 1) / kTW);
  if (tiles == 0) return hipSuccess;
  if (tiles > (1LL << 30)) return hipErrorInvalidValue;
  conv_in_k<false><<<static_cast<unsigned>(tiles), 256, 0, st>>>(x, FrameGlue{}, w_fwd, bias, y, s);
  return hipGetLastError();
}

hipError_t conv3x3_in_frame(const FrameGlue& g, const uint16_t* w_fwd, const float* bias, const Map& y,
                            const Shape& s, hipStream_t st) {
  if (y.c != 32 || y.ld % 8 || y.off % 8 || s.n != 1 || s.h != g.height || s.w != g.width) return hipErrorInvalidValue;
  if (static_cast<long long>(s.h) * s.w * y.ld >= (1LL << 30)) return hipErrorInvalidValue;
  const long long tiles = static_cast<long long>((s.h + kInTH - 1) / kInTH) * ((s.w + kTW - 1) / kTW);
  if (tiles == 0) return hipSuccess;
  const Map none{nullptr, 0, 0, 0};
  conv_in_k<true><<<static_cast<unsigned>(tiles), 256, 0, st>>>(none, g, w_fwd, bias, y, s);
  return hipGetLastError();
}

hipError_t conv3x3_out_frame(const Map& x, const uint16_t* w_fwd, const float* bias, const float* ow, const float* ob,
                             const FrameGlue& g, float tau, float* den, void* final_out, uint32_t mode,
                             float inv_gamma, const Shape& s, uint32_t* tickets, hipStream_t st) {
  if (x.c != 32 || x.ld % 8 || x.off % 8 || !den || s.n != 1 || s.h != g.height || s.w != g.width)
    return hipErrorInvalidValue;
  if ((mode & (kModeFmtRGBA8 | kModeFmtF32)) && !final_out) return hipErrorInvalidValue;
  const long long T = static_cast<long long>(g.tiles_x) * ((g.height + g.tile_h - 1) / g.tile_h);
  if (T * g.P * 16 >= (1LL << 31) || static_cast<long long>(s.h) * s.w * x.ld >= (1LL << 30))
    return hipErrorInvalidValue;
  const Map none{nullptr, 0, 0, 0};
  const OutConv oc{ow, ob, g, tau, den};
  const Map y{nullptr, 32, 0, 32};
  hipError_t e = launch_conv<32, 32, DFB_TH_32_32, false, kEpiFrame>(x, none, w_fwd, bias, y, none, oc, s, tickets, st);
  if (e != hipSuccess) return e;
  frame_display_k<<<blocks(T * g.P, 256), 256, 0, st>>>(g, den, final_out, mode, inv_gamma);
  return hipGetLastError();
}

hipError_t out_conv_fwd(const Map& x, const float* w, const float* b, const float* base, int base_ld, float* out,
                        const Shape& s, hipStream_t st) {
  out_fwd_k<<<blocks(s.pixels(), 256), 256, 0, st>>>(x, w, b, base, base_ld, out, s);
  return hipGetLastError();
}

int out_rows(const Shape& s) { return static_cast<int>((s.pixels() + kOutChunk - 1) / kOutChunk); }

hipError_t out_conv_backward(const Map& x, const float* base, int base_ld, const float* target, const float* w,
                             const float* b, const Map& g, float* bias, float* partial, const Shape& s, hipStream_t st) {
  if (x.c != 32 || x.ld % 8 || x.off % 8 || g.ld % 8 || g.off % 8) return hipErrorInvalidValue;
  const float scale = 2.f / static_cast<float>(s.pixels() * 3);
  out_bwd_k<<<static_cast<unsigned>(out_rows(s)), 256, 0, st>>>(x, base, base_ld, target, w, b, g, bias, partial,
                                                               s.pixels(), scale);
  return hipGetLastError();
}

hipError_t pack_input(const float* in, int in_ld, uint16_t* x, const Shape& s, hipStream_t st) {
  if (reinterpret_cast<uintptr_t>(x) % 16) return hipErrorInvalidValue;
  pack_input_k<<<blocks(s.pixels(), 256), 256, 0, st>>>(in, in_ld, x, s.pixels());
  return hipGetLastError();
}


hipError_t refresh_bf16(const float* w_master, uint16_t* w_fwd, uint16_t* w_dgrad, int ci, int co, hipStream_t st) {
  const int ci_pad = (ci + 7) / 8 * 8;
  refresh_k<<<blocks(9LL * ci_pad * co, 256), 256, 0, st>>>(w_master, w_fwd, w_dgrad, ci, ci_pad, co);
  return hipGetLastError();
}

hipError_t frame_to_input(const FrameGlue& g, float* in6, hipStream_t st) {
  frame_to_input_k<<<blocks(static_cast<long long>(g.width) * g.height, 256), 256, 0, st>>>(g, in6);
  return hipGetLastError();
}


}  // namespace unet
}  // namespace dfb
