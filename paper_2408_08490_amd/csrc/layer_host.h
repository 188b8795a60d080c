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

// Whether a forward launch of `tiles` tiles of 128x128 uses 64x64 ones instead, of which a compute unit holds four (of the large
// ones two).  Up to 320 or so large ones leave compute units with one block or none; from there to a full round they bring in an
// operand half as often as small ones.  In fp32 in front of a ReLU the sums are the fp32 MFMA's, which is the bound, and the small
// tiles' finer rounds count for more.  Outputs of up to 64 columns leave half of a large tile to padding, which fp32 pays for at every
// size, and bf16 until memory bounds both forms.  us, large / small, of a layer's whole forward, outputs wide x tiles:
//   bf16, ReLU, 3 relations of 128 columns: 128 x 300 44.9 / 42.4, x 400 50.7 / 53.1; 264 x 318 37.9 / 37.5; 512 x 280 36.8 / 36.3, x 360 38.7 /
//   40.2; of 256 columns: 256 x 314 58.9 / 56.5, x 400 62.9 / 70.6; 349 x 306 54.5 / 53.4, x 390 58.9 / 66.1.  (Between 200 and 256 large ones, one to
//   a compute unit, are 1.0 to 1.06 times as fast.)  Without it: 256 x 314 31.3 / 31.8, x 470 37.7 / 43.0.
//   fp32, ReLU: 128 x 352 132 / 119; 256 x 314 110 / 89, x 470 123 / 128, x 704 178 / 176, x 1094 285 / 270; 352 x 471 113 / 122, x 1056 262 /
//   238; 512 x 408 106 / 104, x 628 156 / 144, x 1408 304 / 293, x 2188 456 / 463.  Without it: 256 x 314 80.5 / 75.9, x 470 95 / 107; 352 x
//   306 74.0 / 68.8, x 705 132 / 135; 512 x 408 79.6 / 84.7.
//   Up to 64 columns, 3 relations of 128: fp32, ReLU, 64 x 700 173 / 123, x 1500 354 / 255, x 2100 514 / 361; without it 64 x 330 87 / 65, x 1500 285 / 243,
//   32 x 1500 277 / 236; of 256 64 x 960 389 / 347.  bf16, ReLU, 64 x 330 45.7 / 40.8, x 960 103 / 98, x 1500 176 / 178, of 256 64 x 960 230 / 233; without it
//   64 x 960 73 / 68, x 1500 111 / 103.
static inline bool fwd_small_tiles(int dtype, int H, bool relu, int tiles) {
  if (H <= 64) return dtype == HGNN_F32 || tiles < 1000;
  if (dtype == HGNN_F32 && relu) return tiles < 420 || (tiles > 512 && tiles < 2000);
  return tiles < 320;
}

// Column blocks of a backward launch's segments, with tiles of 128 and of 64, and its destination types.
struct BwdCols {
  int c128 = 0, c64 = 0, types = 0;
  void segment(int F) { c128 += (F + 127) / 128; c64 += (F + 63) / 64; }
};
// Whether a backward launch of `tiles` tiles of 128x128, whose products run over rows of G' of `width` scalars, uses 64x64
// ones instead, which are a quarter of the work.  The chip holds 512 of the large ones at a time and 1024 of the small: four small
// blocks of a compute unit cover each other's loads, splitting into planes (fp32) and barriers better than two large ones; what
// speaks for the large ones is that they bring in (and split) an operand half as often, the more the longer the products are.
// Hence the line falls with the width.  (us, large / small, of a layer's whole backward in a loop; columns: of each of the launch's
// segments.)
//   fp32, width 64: 470 tiles 38.8 / 36.9, 1110 70.3 / 62.9, 2928 188 / 174, 5200 265 / 240 (the launch; of 256 columns 243 / 217), half of whose
//   large tiles is padding; 128: 640 67.0 / 52.9, 1335 112 / 106 (96 columns 101.2 /
//   100.9), 1880 155 / 157; 160: 1410 128.1 / 127.5, 1965 188 / 192; 192: 985 98.7 / 93.1, 384 columns 1485 146 / 149; 224: 965 105.2 /
//   106.5; 256: 675 84.6 / 74.4, 830 99.5 / 96.2 (96 columns 91.5 / 92.7), 1025 121 / 123; 320: 685 97.0 / 87.7, 855 113.4 / 111.7; 512: 675
//   126 / 120, 696 127.2 / 123.5, 830 148 / 156.
//   Where a quarter and more of the large tiles' columns is padding, farther out: 192 columns, width 128 1570 113 / 99, 256 1570 165 / 155,
//   512 1570 279 / 272.  And one full round of large tiles is as good as the small ones at widths of 65 to 160 that they pad little: 128
//   columns, width 128 320 40.1 / 40.1; 96 columns 300 36 / 36, 400 39.5 / 41.4; width 160 420 41.4 / 42.2.
//   bf16, width 64: 835 tiles 47.6 / 40.7, 1336 52.5 / 54.7; 128: 545 45.7 / 38.2, 872 49.3 / 47.5, 1336 56 / 61; 256: 648 49.3 / 47.4, 885
//   55.0 / 59.8; 352: 448 49.9 / 47.9, 615 53.2 / 56.2; 512: 320 50.9 / 45.1, 455 52.4 / 51.0, 472 52.3 / 52.2, 650 57.4 / 63.1.
//   Without input gradients (`both` false) a tile's reduction is long, and the slices are cut so that some 640 large tiles are left whatever
//   the rows; beyond, a block has 64 K-steps.  There small ones win to the end of their own round and then lose more.  Large / small tiles, us
//   of the launch, bf16: width 64: 336 47.5 / 37.5, 480 51.4 / 55.0, 544 70.8 / 64.0, 720 160 / 177; 128: 272 49.2 / 38.1, 336 56.7 / 55.5, 400 55.9 / 66.4,
//   624 94.8 / 102; 256: 288 46.2 / 39.4, 352 44.7 / 45.0, 480 51.9 / 59.1, 640 74.2 / 85.1; 349: 288 47.6 / 44.8, 336 52.2 / 55.7, 480 58.4 / 67.5, 912 170 / 254;
//   512: 320 43.9 / 37.2, 384 44.0 / 43.7, 448 48.4 / 52.0, 960 158 / 239.  Of 64 columns, half padding, 128: 400 42.5 / 35.2, 600 67.1 / 57.8;
//   of 192, a quarter, 512 55.7 / 68.1.
//   fp32: 640 and fewer always (512: 448 32.5 / 26.4, 640 48.6 / 30.5); 128: 800 361 / 385, 1008 384 / 477; 256: 800 349 / 376; 320: 912 352 / 357; but 64: 800
//   339 / 231; 160: 1312 516 / 460; 176: 800 344 / 297, 1408 513 / 491; 192 columns, 128: 1200 480 / 444.
static inline bool bwd_small_tiles(int dtype, int tiles, int width, const BwdCols &c, bool both) {
  if (tiles < 256) return true;
  const int padding = 2 * c.c128 - c.c64;   // in blocks of 64 columns, of 2 c128
  const bool padded = 2 * padding >= c.c128;
  if (!both && dtype == HGNN_BF16) return tiles < (padding >= c.c128 || width <= 64 ? 640 : 320);
  if (dtype == HGNN_BF16) return tiles < (width <= 64 ? 1000 : width <= 128 ? 880 : width <= 256 ? 680 : width <= 352 ? 500 : 460);
  if (width <= 64) return true;
  if (padded) return tiles < 1600;
  if (!both) return tiles < (width > 128 && width <= 192 ? 1600 : 700);
  if (width <= 160 && tiles < 512) return c.c128 <= c.types;   // (one column block per row block: its tiles share no operand)
  return tiles < (width <= 160 ? 1350 : width <= 192 ? 1000 : width <= 320 ? 800 : 700);
}

// Rows per slice of the weight-gradient reduction in a launch of `dw_steps` K-steps (over all its tiles) beside
// `other_steps` K-steps of other tiles.  A block's share is 1/640 of the launch's K-steps: a bit over the chip's 512 block
// slots, so that the launch is one long round whose end the shorter blocks fill.  With 64x64 tiles, of which 1024 are resident, it
// is 1/1280 (1/1024 is within 1 % nearly everywhere; fp32, width 512, 160 large tiles 64.7 / 58.8 us, 728 168.5 / 174.1).  Every slice ends with a tile's worth of atomic adds (the chip does about 0.4e12 a second, 40 ns
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
