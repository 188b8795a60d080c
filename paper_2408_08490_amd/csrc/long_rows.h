// Rows of the transpose longer than kLongRow entries (a popular source vertex), in the launches that sum the short ones:
// a whole block takes up to kChunk entries of one row.  Rows of one piece, nearly all of them, are finished there.  The
// blocks of a longer row leave fp32 partial sums, and the one that finishes last adds them up, in the order of the pieces,
// so that the result does not depend on which that is.  The partial sums and the counter go through stores, loads and adds
// of device scope: those of other XCDs see them without a write-back of the L2.
// (As a launch of its own behind the sums, with pieces of 16 entries, the last step was 4 to 8 us of every layer and 27 us of
// the attention variant's largest.)
#pragma once
#include "common.h"
#include "device_types.h"

namespace hgnn {

struct LongPiece {
  int c, beg, n;       // source row, first entry, entries of the piece
  int first, pieces;   // first piece of the row, its pieces
};
__device__ __forceinline__ LongPiece long_piece(const LayerDev &L, int item) {
  LongPiece p;
  p.c = L.chunk_row[item];
  p.beg = L.chunk_beg[item];
  const int j0 = L.cptr[p.c], j1 = L.cptr[p.c + 1];
  p.n = min(kChunk, j1 - p.beg);
  p.first = item - (p.beg - j0) / kChunk;
  p.pieces = (j1 - j0 + kChunk - 1) / kChunk;
  return p;
}

template <int N> struct LongLds {
  float red[4 * 64 * N];
  uint32_t before;   // blocks of the row that finished before this one
};

// Called by all 256 threads of a block.  A row is `nvec` vectors of N floats; 2^l2 (at most 64) lanes share it, so that the
// block holds 256 >> l2 groups.  sum(q, g, groups, acc): adds vector q of the piece's entries g, g + groups, ... to acc;
// done(q, acc): takes vector q of the finished row.  `partial` has a row of `pitch` floats per piece, `count` a zero for
// each.
template <int N, typename Sum, typename Done>
__device__ __forceinline__ void long_row_piece(const LongPiece &p, int item, int l2, int nvec, LongLds<N> &sm, float *partial, int pitch,
                                               uint32_t *count, Sum sum, Done done) {
  const int lanes = 1 << l2, groups = 256 >> l2, col = threadIdx.x & (lanes - 1), g = threadIdx.x >> l2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // adds up the groups' sums; the first `lanes` threads of the block get the result
  auto meet = [&](float (&acc)[N]) {
    for (int o = lanes; o < 64; o <<= 1) {
#pragma unroll
      for (int k = 0; k < N; ++k) acc[k] += __shfl_xor(acc[k], o);
    }
    __syncthreads();
    if (lane < lanes) {
#pragma unroll
      for (int k = 0; k < N; ++k) sm.red[(wave * 64 + lane) * N + k] = acc[k];
    }
    __syncthreads();
    if ((int)threadIdx.x >= lanes) return false;
#pragma unroll
    for (int w = 1; w < 4; ++w)
#pragma unroll
      for (int k = 0; k < N; ++k) acc[k] += sm.red[(w * 64 + lane) * N + k];
    return true;
  };
  for (int q0 = 0; q0 < nvec; q0 += lanes) {
    const int q = q0 + col;
    float acc[N];
#pragma unroll
    for (int k = 0; k < N; ++k) acc[k] = 0.f;
    if (q < nvec) sum(q, g, groups, acc);
    if (!meet(acc) || q >= nvec) continue;
    if (p.pieces == 1) {
      done(q, acc);
    } else {
      unsigned long long *o = reinterpret_cast<unsigned long long *>(partial + (int64_t)item * pitch + q * N);
#pragma unroll
      for (int k = 0; k < N; k += 2)
        __hip_atomic_store(o + k / 2, (unsigned long long)__float_as_uint(acc[k]) | ((unsigned long long)__float_as_uint(acc[k + 1]) << 32),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (p.pieces == 1) return;
  if (wave == 0) {   // the wavefront that stored: its stores are at the coherence point before the count goes up
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0) sm.before = __hip_atomic_fetch_add(count + p.first, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (sm.before != (uint32_t)(p.pieces - 1)) return;
  for (int q0 = 0; q0 < nvec; q0 += lanes) {
    const int q = q0 + col;
    float acc[N];
#pragma unroll
    for (int k = 0; k < N; ++k) acc[k] = 0.f;
    if (q < nvec) {
      for (int j = g; j < p.pieces; j += groups) {
        const unsigned long long *o = reinterpret_cast<const unsigned long long *>(partial + (int64_t)(p.first + j) * pitch + q * N);
        unsigned long long v[N / 2];
#pragma unroll
        for (int k = 0; k < N / 2; ++k) v[k] = __hip_atomic_load(o + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int k = 0; k < N; k += 2) {
          acc[k] += __uint_as_float((uint32_t)v[k / 2]);
          acc[k + 1] += __uint_as_float((uint32_t)(v[k / 2] >> 32));
        }
      }
    }
    if (meet(acc) && q < nvec) done(q, acc);
  }
}

}  // namespace hgnn
