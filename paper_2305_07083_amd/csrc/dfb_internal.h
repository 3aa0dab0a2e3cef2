// Internal interface between the host runtime (dfb_runtime.hip) and the
// gfx950 kernels (dfb_kernels.hip).  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/dfb.h"

namespace dfb {

// Layers per tile handled by the register sort; above it, the row sort and
// the workgroup-wide LDS sort take over.
constexpr int kRegMax = 32;
// Layers per tile handled by the row sort (16 lanes of a wave sort a pixel in
// registers); tiles with more, up to kMaxLayers, take the LDS sort.
// 512: their 32 keys a lane and 74 KB of alphas still leave two workgroups
// to a compute unit.
constexpr int kDeepMax = 512;
constexpr int kDeepThreads = 512;
constexpr int kDeepPx = 32;  // pixels of a row-sort group: one 128-byte line of an fp32 plane
// Work queue: the work list is dealt round-robin to kQueues counters, each
// in its own 4 KB page, served first by the workgroups with the same index
// mod kQueues, so same-address atomics do not serialise the whole chip.
// Each counter has kSlots per-frame slots used as a ring: frame f counts in
// slot f mod kSlots and clears slot (f + kSlots/2) mod kSlots, which no
// frame in flight uses, so nothing is reset between frames.  A ring is the
// kQueues counter pages and one page more; kFinishWord words into a page lie
// the slots of its "workgroups finished" counter (the counters' own, then the
// one that counts the counters).  A frame runs up to three launches over the
// same work list -- the tiles of more than kDeepMax layers, those of more
// than kRegMax, then the rest, which counts its finished workgroups -- each
// with a ring of its own; after the rings comes one page holding the
// FrameState below.
constexpr int kQueues = 16;
constexpr int kQueueStride = 1024;  // 4-byte counters between queues
constexpr int kSlots = 64;
constexpr int kFinishWord = 512;    // in a page, so a ticket and a finish counter share no line
constexpr int kRingWords = (kQueues + 1) * kQueueStride;
constexpr int kRings = 3;
constexpr int kQueueWords = kRings * kRingWords + kQueueStride;  // the whole allocation, in u32

// Per-handle frame state in device memory.  Kernels read it at their start
// and the last workgroup of a frame advances it, so a launch carries no
// per-frame value in its arguments and one captured frame can be replayed
// as every later frame.
struct FrameState {
  uint32_t seq;    // frames so far: selects the counter slot
  int32_t n_acc;   // frames folded into the running mean since the reset
};
// Ring r (0: the register-path launch, 1: the LDS sort's, 2: the row sort's)
// and the frame state inside a queue allocation.
inline uint32_t* ring_of(uint32_t* queue_base, int r) { return queue_base + r * kRingWords; }
// Units that counter s of S holds of n_work units dealt in blocks of B.
__host__ __device__ inline int queue_units(int n_work, int B, int S, int s) {
  const int nb = (n_work + B - 1) / B;
  const int cnt = s < nb ? (nb - s + S - 1) / S : 0;
  int n = cnt * B;
  if (cnt > 0 && s + (cnt - 1) * S == nb - 1 && n_work % B) n -= B - n_work % B;  // partial last block
  return n;
}
inline FrameState* state_of(uint32_t* queue_base) {
  return reinterpret_cast<FrameState*>(queue_base + kRings * kRingWords);
}
constexpr int kMaxLayers = 4096;
// Largest LDS budget of the LDS sort for keys (u64) and weights (f32);
// the host passes 64, 96 or 112 KB depending on the frame's largest tile.
constexpr int kBigLdsBytes = 112 * 1024;

enum ModeBits : uint32_t {
  kModeAccumulate = 1u,     // fold into the running mean + per-tile variance
  kModeKeepFinished = 2u,   // store the finished f32 tile
  kModeKeepOrder = 4u,      // store the per-pixel sorted order (debug)
  kModeFmtRGBA8 = 8u,       // display: RGBA8
  kModeFmtF32 = 16u,        // display: RGBA f32
  kModeGamma = 32u,         // colour ^ (1/gamma) before quantising
};

// A tile of a launch's list: one read takes a workgroup from a list position to
// its tile's layers.  With a list of units and the offsets apart it took two
// dependent ones, about 1 us of every unit: 1024x1024, every frame a new
// layout: 51 -> 48 us, small frames 20.4 -> 18.7.
struct alignas(16) TileRec {
  int32_t tile, off, layers, pad;
};

// Everything one frame launch needs besides the three read-only tables,
// which are separate __restrict__ kernel arguments so that their uniform
// reads become scalar loads:
//   tile_off   [n_tiles + 1] CSR offsets into layer_off
//   layer_off  [n_layers] element offset of each layer's block (block*5*P);
//              per tile ordered by source id
//   recs       [n_tiles] the tiles, most layers first; unit i of a launch is
//              piece i % units-per-tile of the tile at position
//              i / units-per-tile.  Null: the tiles in their own order
// Passed by value; nothing in it changes from frame to frame while the layer
// table, the fragment buffer and the launch shape stay the same.
struct FrameArgs {
  const void* frag;            // fragment blocks (caller's buffer)
  uint32_t* queue;             // this launch's ring
  uint32_t* rings;             // all kRings rings (the frame's last launch recycles a slot of each)
  FrameState* state;           // the frame state (shared by the frame's launches)
  int32_t one_each;            // no counter holds more units than workgroups start on it: no tickets
  int32_t slot, clear_slot;    // set by the kernel from FrameState::seq
  int32_t n_queues;            // counters in use: min(kQueues, grid)
  int32_t queue_block;         // consecutive work-list positions per counter block (units per tile)
  int32_t n_work;
  int32_t list_end;            // set by the kernel: no unit from here on is this launch's
  int32_t width, height, tiles_x, n_tiles;
  int32_t tile_w, tile_h, P;
  int32_t work_w, work_h, subs_x, subs_per_tile, work_px;
  int32_t work_shift;          // log2(work_w) if a power of two, else -1
  int32_t big_lds;             // LDS bytes for keys + weights of the LDS sort
  int32_t vec_ok;              // 16-byte plane loads possible (alignment, work_w, tile_w)
  int32_t deep_subs;           // row-sort launch: units (groups of kDeepPx pixels) per tile, else 0
  int32_t max_run;             // units a draw takes at most (the row sort's; else 1)
  int32_t deep_layers;         // row-sort launch: layers its LDS holds
  int32_t quad_ok;             // 4-pixel plane loads are aligned: the row sort can run
  int32_t big_min;             // LDS sort: it takes the tiles of more layers than this
  float bg[4];
  const float* bg_image;       // [n_tiles][P][4] per-pixel background, or null
  float inv_gamma;
  uint32_t mode;
  int32_t n_acc;               // set by the kernel: accumulation id after this frame
  float inv_n;                 // set by the kernel: 1 / n_acc
  float* finished;             // [n_tiles][P][4]
  float* accum;                // [n_tiles][P][4]
  float* m2;                   // [n_tiles][3][P]
  float* tile_var;             // [n_tiles]
  float* var_partial;          // [n_tiles * subs_per_tile] M2 sum of each unit (accumulating frames)
  float* deep_partial;         // [n_tiles * deep_subs] the same of the row-sort units
  void* final_out;             // RGBA8 uint32[n_tiles][P] or float4[n_tiles][P]
  uint16_t* order;             // [n_layers][P]
};

struct AccumArgs {
  const float* finished;
  float* accum;
  float* m2;
  float* tile_var;
  void* final_out;
  int32_t width, height, tiles_x, n_tiles, tile_w, tile_h, P;
  float inv_gamma;
  uint32_t mode;
  const FrameState* state;     // n = state->n_acc + 1 (advanced by a separate launch)
};

struct VarianceArgs {
  const float* var_partial;    // [n_tiles * subs_per_tile]
  const float* deep_partial;   // [n_tiles * deep_subs]: the tiles of kRegMax + 1 .. kDeepMax layers
  const int32_t* tile_off;
  int32_t deep_subs;           // 0: the frame has no such tiles
  float* tile_var;             // [n_tiles]
  int32_t n_tiles, subs_per_tile, tiles_x, width, height, tile_w, tile_h;
  const FrameState* state;     // n = state->n_acc (already advanced by the frame kernel)
};

struct ValidateArgs {
  const void* frag;
  const int64_t* layer_off;
  int32_t n_layers, P;
  uint32_t* bad;   // set to 1 if a NaN depth is seen
};

// What the denoiser needs from a compositor handle: its accumulation.
struct FrameGlue {
  const float* accum;      // [T][P][4] running mean
  const float* tile_var;   // [T]
  const FrameState* state; // n = state->n_acc
  int width, height, tiles_x, tile_w, tile_h, P;
};
struct FrameView {
  FrameGlue glue;
  void* final_out;         // display buffer (or null for NONE)
  float* denoised;         // [T][P][4] (allocated on request)
  uint32_t display_mode;   // kModeFmt* | kModeGamma
  float inv_gamma;
  hipStream_t stream;
};
// Fails with DFB_ERR_STATE unless at least one frame has been accumulated.
dfb_status frame_view(dfb_ctx* h, FrameView* out, bool want_denoised);

// The persistent frame kernel for a fragment dtype, register-sort capacity
// and tile operation (dfb_tile_op).  dtype: 0 f32, 1 f16.  kcap 8, 16 or 32:
// the per-pixel sort of tiles with at most kcap layers in registers (tiles
// with more are left to the other launches); kcap 0 (ALPHA_BLEND only): the
// workgroup-wide LDS sort of the tiles with more than kDeepMax layers, others
// left alone.
const void* frame_kernel(int dtype, int kcap, int op);
// The row sort of the tiles with kRegMax + 1 .. kDeepMax layers
// (ALPHA_BLEND), others left alone, and its dynamic LDS; kDeepThreads lanes.
const void* deep_kernel(int dtype, int max_layers);
size_t deep_lds_bytes(int max_layers);
// Layers of a row-sort tile its LDS is sized for (even: what follows stays 16-byte aligned).
inline int deep_layers(int max_layers) { return ((max_layers < kDeepMax ? max_layers : kDeepMax) + 1) & ~1; }
// Largest-remainder assignment of extra samples (host; dfb_assign_samples_host).
dfb_status assign_samples(const float* variance, int32_t n_tiles, int64_t extra, int32_t* counts);
const void* accumulate_kernel();
const void* tile_variance_kernel();
// One thread: state->n_acc = value (value >= 0), or += 1 (value < 0).
const void* state_kernel();
// (uint32_t* p, uint32_t v, int64_t n): p[0..n) = v, any grid.
const void* fill_u32_kernel();
// (const uint32_t* src, uint32_t* dst, int64_t n): dst[0..n) = src[0..n), any grid.
const void* copy_u32_kernel();
// (const int32_t* tile_off, int32_t n_tiles, TileRec* recs): the longest-first
// list, one workgroup of kLptThreads lanes.
const void* lpt_work_kernel();
constexpr int kLptThreads = 1024;
const void* validate_kernel(int dtype);

// LDS budget of the LDS sort for a frame whose largest tile has
// max_layers layers, and the dynamic LDS bytes a frame launch needs (kcap as
// for frame_kernel).
int big_lds_bytes(int max_layers);
size_t frame_lds_bytes(int kcap, int threads, int max_layers, int big_lds);

}  // namespace dfb
