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

// Whether a backward launch of `tiles` tiles of 128x128, whose products run over rows of G' of `width` scalars, uses 64x64
// ones instead.  The chip holds 512 of the large ones at a time and 768 of the small, which are a quarter of the work.
// Below 256 large ones compute units stay empty.
// fp32 tiles are split into planes on the way to LDS, and three small blocks of a compute unit cover each other's splitting,
// loads and barriers better than two large ones; what speaks for the large ones is that an operand is split half as often.
// They win where their rounds are nearly full (us, large -> small): 352 tiles 30 -> 29, 364 47 -> 37, 624 38 -> 34,
// 664 68 -> 57, but 496 34 -> 38, 936 98 -> 108, 1044 116 -> 135, 1192 222 -> 276.
// bf16: small ones where a launch of one round has short products (484 tiles of width 128 23 -> 17, 424 of 256 32 -> 29,
// 360 of 256 31 -> 29, but 400 of 512 33 -> 37, 756 of 264 39 -> 51).
static inline bool bwd_small_tiles(int dtype, int tiles, int width) {
  if (tiles < 256) return true;
  if (dtype == HGNN_BF16) return tiles < 512 && width <= 256;
  return tiles < 384 || (tiles > 512 && tiles < 768);
}

// Rows per slice of the weight-gradient reduction in a launch of `dw_steps` K-steps (over all its tiles) beside
// `other_steps` K-steps of other tiles.  A block's share is 1/640 of the launch's K-steps (1/1280 with 64x64 tiles, of
// which twice as many are resident): a bit over the chip's block slots, so that the launch is one long round whose end
// the shorter blocks fill.  Every slice ends with a tile's worth of atomic adds (the chip does about 0.4e12 a second, 40 ns
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
