// What the host sides of the layer variants share (api.cpp: mean aggregation and the entry points; attn_layer.cpp).
#pragma once
#include "common.h"

namespace hgnn {

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline int esize(int dtype) { return dtype == HGNN_BF16 ? 2 : 4; }

// Waits for the host build and fills the device-side view of one layer's index arrays.
hgnn_status layer_dev(hgnn_ctx *ctx, hgnn_graph *g, int32_t layer, LayerDev &D);

// Makes `s` wait for the graph's upload.  Once the upload is known to have finished no stream has to wait any more (an
// unfinished event costs some 10 us per wait, and a step takes four or more).  Which stream waited before says nothing: a
// handle does not identify a stream (hipStreamPerThread names another one in every thread; a destroyed stream's may come
// again), and a wait that went into a captured graph orders nothing outside it.
static inline hipError_t wait_upload(hgnn_graph *g, hipStream_t s) {
  if (g->uploaded.load(std::memory_order_acquire)) return hipSuccess;
  if (hipPeekAtLastError() == hipSuccess) {   // "not ready" is left as the thread's last error, which is then taken back
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;   // the query may run while a stream is being captured
    const bool exchanged = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    const hipError_t e = hipEventQuery(g->ready);
    if (e != hipSuccess) (void)hipGetLastError();
    if (exchanged) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e == hipSuccess) {
      g->uploaded.store(true, std::memory_order_release);
      return hipSuccess;
    }
  }
  return hipStreamWaitEvent(s, g->ready, 0);
}

// While alive, the launches made on this thread are timed if the probe selects (kernel, layer).
struct Probe {
  bool active = false;
  Probe(hgnn_ctx *c, int kernel, int layer, bool enabled = true);
  ~Probe();
};

// The attention variant's side of the layer entry points.  It registers itself when the library is loaded, so that the
// host runtime links without any device code of the variant.
struct AttnVariant {
  hgnn_status (*workspace)(hgnn_ctx *, hgnn_graph *, int32_t layer, const hgnn_layer_params *, size_t *saved_bytes, size_t *scratch_bytes);
  hgnn_status (*fwd)(hgnn_ctx *, void *stream, hgnn_graph *, int32_t layer, const hgnn_layer_params *, const void *x, void *h, void *saved,
                     size_t saved_bytes, void *scratch, size_t scratch_bytes);
  hgnn_status (*bwd)(hgnn_ctx *, void *stream, hgnn_graph *, int32_t layer, const hgnn_layer_params *, const void *x, const void *h_out,
                     const void *saved, const void *grad_h, void *grad_x, const hgnn_layer_grads *, void *scratch, size_t scratch_bytes);
  hgnn_status (*launch_count)(hgnn_ctx *, hgnn_graph *, int32_t layer, const hgnn_layer_params *, int32_t *fwd, int32_t *bwd);
};
AttnVariant &attn_variant();

// Column blocks of a backward launch's segments, with tiles of 128 and of 64, and its destination types.
struct BwdCols {
  int c128 = 0, c64 = 0, types = 0;
  void segment(int F) { c128 += (F + 127) / 128; c64 += (F + 63) / 64; }
};
// Whether a backward launch of `tiles` tiles of 128x128, whose products run over rows of G' of `width` scalars, uses 64x64
// ones instead, which are a quarter of the work.  The chip holds 512 of the large ones at a time and 768 of the small.  Below 256
// large tiles compute units stay empty.  (Figures: us, large / small, of a layer's whole backward in a loop.)
// fp32 tiles are split into planes on the way to LDS.  Three small blocks of a compute unit cover each other's splitting, loads
// and barriers better than two large ones; what speaks for the large ones is that an operand is split half as often.
//   Up to 384 large tiles, one or two to a compute unit, small ones win with long products (width 176, 312 tiles 44.0 / 41.3;
//   width 256, 324 47.8 / 43.0) and where more than a quarter of the large tiles' columns is padding (64 columns, width 128, 320
//   32.5 / 27.4; width 64, 320 34.0 / 32.3), not otherwise (width 128: 384 columns 300 35.3 / 37.3, 6 x 128 columns 324 38.1 /
//   40.5, 96 columns 304 35.6 / 38.8, 192 columns 352 34.5 / 36.0; width 160 348 37.6 / 40.3) except with one column block per
//   row block, whose tiles share no operand (128 columns of each type, width 128: 308 66.9 / 66.6, 378 72.8 / 71.3).
//   From there to a full round of 512 mostly large ones do (width 160 504 42.8 / 44.7; 384 columns, width 128 480 42.2 / 45.8).
//   In a second round that is not full small ones win up to 768 (width 128, 600 58.5 / 48.9, 750 65.0 / 57.8; width 320, 760 99.3 /
//   95.4), with longer products up to 700 (width 352, 636 100.0 / 91.9, 702 105.2 / 104.0, 750 107.4 / 111.2; width 512, 640
//   125.5 / 116.6, 748 140 / 151) unless a quarter is padding (192 columns, width 512, 744 126.7 / 115.6).
// bf16: small ones where a launch of one round of large tiles has products of at most 256 (width 128: 300 44.5 / 30.6, 476
// 46.2 / 39.4; width 256: 400 46.7 / 43.3, 504 47.9 / 47.7; width 352: 480 50.7 / 52.7).
static inline bool bwd_small_tiles(int dtype, int tiles, int width, const BwdCols &c) {
  if (tiles < 256) return true;
  if (dtype == HGNN_BF16) return tiles < 512 && width <= 256;
  const int padding = 2 * c.c128 - c.c64;   // in blocks of 64 columns, of 2 c128
  if (tiles < 384) return width > 160 || width <= 64 || 2 * padding > c.c128 || c.c128 <= c.types;
  return tiles > 512 && tiles < (width <= 320 || 2 * padding >= c.c128 ? 768 : 700);
}

// Rows per slice of the weight-gradient reduction in a launch of `dw_steps` K-steps (over all its tiles) beside
// `other_steps` K-steps of other tiles.  A block's share is 1/640 of the launch's K-steps: a bit over the chip's 512 block
// slots, so that the launch is one long round whose end the shorter blocks fill.  With 64x64 tiles it is 1/1280, which is more
// than the 768 of them that are resident: shares of 1/832 and 1/768 were up to a quarter faster in launches of some 500 small
// tiles and up to 5 % slower in larger ones with long products (fp32, 128 columns, us at 1/1280, 1/832, 1/768: width 512, 320
// large tiles 39.5, 29.8, 29.4, but 640 91.7, 96.3, 91.4; width 128, 304 27.4, -, 24.8).  Every slice ends with a tile's worth of atomic adds (the chip does about 0.4e12 a second, 40 ns
// of all of it per 128x128 tile), hence the least number of K-steps: 32 of bf16 (8 measured 9 us worse on 4096 rows of
// 512 x 349); an fp32 K-step is several times as long (1.7 us of a compute unit's matrix cores per 128x128 tile), which
// both keeps the adds cheap beside it and makes long slices a serial chain (64 K-steps in one block were 183 us of a
// 500 us step).
static inline int dw_slice_rows(int dtype, int edge, int64_t dw_steps, int64_t other_steps) {
  const int bk = dtype == HGNN_BF16 ? 64 : 32, least = dtype == HGNN_BF16 ? (edge == 64 ? 8 : 32) : 4;
  const int64_t share = edge == 64 ? 1280 : 640, steps = (dw_steps + other_steps + share - 1) / share;
  return bk * (int)(steps < least ? least : steps > 64 ? 64 : steps);
}

}  // namespace hgnn
