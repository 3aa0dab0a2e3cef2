// Internal interface between the denoiser runtime (unet_runtime.hip) and its
// gfx950 kernels (unet_kernels.hip).  Not part of the C ABI.
//
// Layouts: activations NHWC; bf16 maps are stored as uint16 bit patterns;
// a map may be a channel slice of a wider buffer (row stride `ld`, first
// channel `off`).  conv3x3 weights (f32 master) are [3][3][ci][co]; the
// kernels read two bf16 copies: fwd [9][co][ci] and dgrad [9][ci][co].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfb_internal.h"

namespace dfb {
namespace unet {

struct Map {          // bf16 NHWC map (or a channel slice of one)
  uint16_t* p;
  int ld, off, c;     // row stride (channels), first channel, channels
};
struct Shape {
  int n, h, w;        // batch, height, width
  __host__ __device__ long long pixels() const { return static_cast<long long>(n) * h * w; }
};

// y = bf16(relu(conv3x3(x') + b)) at the output shape s, where x' = x, or
// with `up` the nearest-neighbour 2x up-sampling of x (x at s/2).  x channels
// must be a multiple of 8; s.h and s.w even with `up` or `pool`.  With `pool`,
// also pool = bf16(2x2 average of y) at s/2.  With `x2`, the input is the
// channel concatenation of x and x2 (x.c a multiple of 32, x2.ld == x.ld):
// two maps that are each written with full 64- or 128-byte pixel rows.
// `tickets`: kTicketWords words, zero between launches (each leaves them so),
// for launches of one stream at a time.
constexpr int kTicketWords = 8 * 32;
hipError_t conv3x3_fwd(const Map& x, const uint16_t* w_fwd, const float* bias, const Map& y,
                       const Shape& s, uint32_t* tickets, hipStream_t st, bool up = false,
                       const Map* pool = nullptr, const Map* x2 = nullptr);
// The data gradient of a conv3x3 (ci input channels, a multiple of 32; g its
// gated output gradient at shape s), carried through to the gated output
// gradient o.g of the layer that made its input: g' = bf16(dx' * (y > 0)), y
// that layer's output.  dx' is dx itself; with kUp (the input was 2x
// up-sampled) the 2x2 sums of dx, at s / 2; with kPool (it was 2x2 pooled)
// o.skip + dx / 4 at 2 s.  With kSame, channels from 32 o.split on are the
// skip of a concatenation: their dx goes to o.skip, ungated.  partial[row][c],
// c < o.g.c, over the conv_tiles(s, ci) rows, sums to the layer's bias gradient
// in f32.
enum class Adjoint { kSame, kUp, kPool };
struct TileOut {
  Map y;               // forward: the output; gradient: the activation that gates
  Map g, pool;
  float* skip;         // [pixel][skip_ld]
  int skip_ld, split;
  float* partial;
};
int conv_tiles(const Shape& s, int co);
hipError_t conv3x3_bwd(const Map& g, const uint16_t* w_dgrad, int ci, Adjoint adj, const TileOut& o, const Shape& s,
                       hipStream_t st);

// Weight gradients of the 12 conv3x3 layers, one launch: partial sums of
// dw[9][ci][co] = sum_p x[p + tap] * g[p] over `chunks` runs of pixel tiles.
constexpr int kConvLayers = 12;
struct WgradLayer {
  const uint16_t* x;   // input map [source pixels][xld], its xc channels first (16-byte aligned)
  const uint16_t* g;   // gated output gradient [pixels][co]
  int xld, xc, co;
  int up;              // x is the map the layer's input is 2x up-sampled from
  Shape s;             // output shape
  int cb, ob;          // 32-channel slices of c_in and c_out a workgroup takes (1 or 2)
  int cig, cog;        // such groups
  int tiles, chunks, first_wg;
  size_t part;         // first float of the layer's partial sums
};
struct WgradPlan {
  WgradLayer l[kConvLayers];
  int n_wg;
};
int wgrad_chunks(int layer, long long tiles);
long long wgrad_tiles(const Shape& s);
size_t wgrad_floats(const WgradLayer& L);  // of its partial sums
hipError_t conv3x3_wgrad(const WgradPlan& plan, float* partial, hipStream_t st);

// The sums of every gradient's partials, Adam, and the bf16 weight copies.
struct UpdateLayer {
  int cb, ob, cig, cog, chunks, first_block;
  int ci, ci_pad, co;
  int off_w;           // first weight in the parameter vector
  size_t part;
  uint16_t *wf, *wd;   // forward [9][co][ci_pad] and data-gradient [9][ci_pad][co] copies
};
struct BiasPart {      // n columns (parameters) of `rows` partial rows
  int first, n, rows, param;
  size_t part;
};
struct UpdatePlan {
  UpdateLayer l[kConvLayers];
  BiasPart bias[kConvLayers + 1];  // the layers' biases, then the output conv's 99 parameters and the loss sum
  int conv_blocks;
};
struct AdamArgs {
  float *w, *g, *m, *v, *loss;
  float lr, b1, b2, eps, c1, c2;
  int update;          // 0: gradients and loss only
};
int update_blocks(const UpdateLayer& L);
hipError_t update_params(const UpdatePlan& plan, const float* partial, const AdamArgs& a, hipStream_t st);

// The first conv3x3 (8 input channels -> 32, ReLU, bf16) with the nine
// taps packed into a 72-deep contraction, reading the packed bf16 input x
// (x.c == 8).
hipError_t conv3x3_in_fwd(const Map& x, const uint16_t* w_fwd, const float* bias, const Map& y, const Shape& s,
                          hipStream_t st);
// out[p][c] = base[p][c] + b[c] + sum_i x[p][i] w[i][c]   (c < 3, f32)
hipError_t out_conv_fwd(const Map& x, const float* w, const float* b, const float* base,
                        int base_ld, float* out, const Shape& s, hipStream_t st);
// out as out_conv_fwd's, dout = 2 (out - target) / count, g = bf16(dout w^T *
// (x > 0)), the gated output gradient of the conv that made x (32 channels);
// over out_rows rows, bias[row][32] sums to that conv's bias gradient and
// partial[row] to {dw[c][3], db[3], sum (out - target)^2}.
hipError_t out_conv_backward(const Map& x, const float* base, int base_ld, const float* target, const float* w,
                             const float* b, const Map& g, float* bias, float* partial, const Shape& s, hipStream_t st);
int out_rows(const Shape& s);

// bf16 input [p][8] from f32 [p][in_ld] (first 6 channels), channels 6,7 zero.
hipError_t pack_input(const float* in, int in_ld, uint16_t* x, const Shape& s, hipStream_t st);

// The bf16 copies of a layer's master weights.
hipError_t refresh_bf16(const float* w_master, uint16_t* w_fwd, uint16_t* w_dgrad, int ci, int co,
                        hipStream_t st);

// Compositor glue: NHWC denoiser input from tile-major mean / tile variance.
using dfb::FrameGlue;
hipError_t frame_to_input(const FrameGlue& g, float* in6, hipStream_t st);
// conv3x3_in_fwd reading that input straight from the frame (one image of
// the frame's size), without materialising it.
hipError_t conv3x3_in_frame(const FrameGlue& g, const uint16_t* w_fwd, const float* bias, const Map& y,
                            const Shape& s, hipStream_t st);
// The last conv3x3 (32 -> 32, ReLU, bf16) fused with the output conv and
// written into the frame: with out[p][c] = mean[p][c] + ob[c] + sum_i y[p][i]
// ow[i][c] (y the conv's bf16 output, not stored), den[e] = (out, mean
// alpha), or the mean where the tile falls back
// (n >= 2 and variance > tau); padding pixels of ragged edge tiles get the
// mean; then the display value of every pixel in final_out by mode
// (kModeFmtRGBA8 / kModeFmtF32, kModeGamma).  den is required; final_out
// when mode has a format.
hipError_t conv3x3_out_frame(const Map& x, const uint16_t* w_fwd, const float* bias, const float* ow, const float* ob,
                             const FrameGlue& g, float tau, float* den, void* final_out, uint32_t mode,
                             float inv_gamma, const Shape& s, uint32_t* tickets, hipStream_t st);

}  // namespace unet
}  // namespace dfb
