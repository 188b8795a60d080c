// Work of one block on a list of weight transposes (TransposeJobs): block b of nb takes the 32x32 tiles b, b + nb, ...
// of all jobs.  `tile` is a 32x33 LDS buffer of the calling kernel; every thread of the (256-thread) block calls this.
#pragma once
#include "common.h"
#include "device_types.h"

namespace hgnn {

// A launch in which tj.blocks blocks transpose beside others: tb, the block's place among those (outside 0 .. tj.blocks - 1: it
// is none of them), and b, its place among the others.  In front the transposes' weights, which come from HBM, the longest chain
// of loads in the launch, are under way from the start; behind, the transposes fill the places that become free instead of
// holding those of blocks with more to do.
// Behind is mostly the better of the two from a chip's worth of blocks on (2048 of 256 threads) in the aggregation of one width.
// Forward of a layer, us, in front / behind: 108 relations, two layers 57.0 / 54.6; 8 relations, 128 features in bf16, 888 blocks
// 31.3 / 31.3, 1688 34.5 / 34.8, 3288 49.1 / 48.4, with 512 outputs 8576 130.9 / 129.3; read from the stores 2688 48.9 / 48.3; rows of
// 3 KB, of whose blocks the chip holds 1024, 1752 53.0 / 51.5 and 2552 77.2 / 76.6 in bf16, but 1280 of them in fp32, 1476 76.7 /
// 77.2.  Not always: 10 types, 256 features in bf16, rows of 7 edges, 3500 blocks 64.0 / 66.6; 30 relations, 64 features, rows of 2
// edges, 8248 blocks 60.9 / 61.6.
// Ragged widths keep them in front: 96 and 128 features in bf16, 2280 blocks 34.3 / 35.3, 3280 38.6 / 39.1; in fp32, 2140 45.0 / 45.6;
// 32 and 384, 3484 44.1 / 45.1; 10 types of 32 to 384, two layers of 72 and 242 outputs 111.9 / 112.3, of 424 and 75 160.0 / 159.1.
// (With many relations behind would be the better: 104 of ragged widths, 1173 destinations, 34.1 / 32.6.)
struct JobSplit {
  int tb, b;
  __device__ __forceinline__ explicit JobSplit(const TransposeJobs &tj) {
    const bool first = gridDim.x <= 2048;
    tb = first ? (int)blockIdx.x : (int)blockIdx.x - ((int)gridDim.x - tj.blocks);
    b = first ? (int)blockIdx.x - tj.blocks : (int)blockIdx.x;
  }
  __device__ __forceinline__ bool transposes(const TransposeJobs &tj) const { return tb >= 0 && tb < tj.blocks; }
};

template <typename T>
__device__ __forceinline__ void transpose_jobs_block(const TransposeJobs &tj, int b, int nb, T (*tile)[33]) {
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  const int total = tj.tile_off[tj.n];
  const int H = tj.H, tiles_h = (H + 31) / 32;
  for (int tl = b; tl < total; tl += nb) {
    const int job = wave_find(tj.tile_off, tj.n, tl);
    const int local = tl - tj.tile_off[job];
    const int F = tj.F[job];
    const T *w = reinterpret_cast<const T *>(tj.w[job]);
    T *out = reinterpret_cast<T *>(tj.out) + (int64_t)tj.off4[job] * 4;
    const int f0 = (local / tiles_h) * 32, h0 = (local % tiles_h) * 32;
    for (int i = ty; i < 32; i += 8) {
      const int f = f0 + i, h = h0 + tx;
      if (f < F && h < H) tile[i][tx] = w[(int64_t)f * H + h];
    }
    __syncthreads();
    for (int i = ty; i < 32; i += 8) {
      const int h = h0 + i, f = f0 + tx;
      if (f < F && h < H) out[(int64_t)h * F + f] = tile[tx][i];
    }
    __syncthreads();
  }
}

}  // namespace hgnn
