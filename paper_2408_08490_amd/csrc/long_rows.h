// Rows of the transpose longer than kLongRow entries (a popular source vertex), in the launches that sum the short ones:
// a whole block, or one wavefront of it (long_rows_by_wave), takes up to kChunk entries of one row.  Rows of one piece,
// nearly all of them in a sampled batch, are finished there.  The pieces of a longer row leave fp32 partial sums, and the one
// that finishes last adds them up, in the order of the pieces, so that the result does not depend on which that is.  The
// partial sums and the counter go through stores, loads and adds of device scope: those of other XCDs see them without a
// write-back of the L2.
// (As a launch of its own behind the sums, with pieces of 16 entries, the last step was 4 to 8 us of every layer and 27 us of
// the attention variant's largest.)
#pragma once
#include <type_traits>

#include "common.h"
#include "device_types.h"

namespace hgnn {

struct LongPiece {
  int c, beg, n;            // source row, first entry, entries of the piece
  int first, pieces, row;   // place of the row's first piece among the partial sums, its pieces, its first chunk
};
// `halves`: 1 where a chunk of kChunk entries is two pieces, else 0
__device__ __forceinline__ LongPiece long_piece(const LayerDev &L, int item, int halves = 0) {
  const int chunk = item >> halves, size = kChunk >> halves;
  LongPiece p;
  p.c = L.chunk_row[chunk];
  const int j0 = L.cptr[p.c], j1 = L.cptr[p.c + 1], beg = L.chunk_beg[chunk];
  p.beg = beg + (item - (chunk << halves)) * size;
  p.n = min(size, j1 - p.beg);   // none behind a row's last entry
  p.row = chunk - (beg - j0) / kChunk;
  p.first = p.row << halves;
  p.pieces = (j1 - j0 + size - 1) >> (31 - __clz(kChunk) - halves);
  return p;
}

// Whether a wavefront takes a piece instead of a block, four to a block.  As long as the chip gets through the blocks in a round
// or two (it holds 2048) four wavefronts are done sooner than one, with a popular row's many pieces above all.  With more, in a
// batch of dense neighbourhoods, what counts is how many pieces are in flight, and a piece of narrow rows has too little work for
// a block (of 17 entries of 2 lanes it uses an eighth).  Rows of more than 16 lanes stay with the block: they give it enough to
// do, and a wavefront would add up 64 entries and more one after the other.  us, a block / a wavefront per piece, rows x entries: 2
// lanes, 20000 x 17 43 / 15, 4000 x 200 37 / 13, 1500 x 17 7.1 / 5.0, 200 x 128 5.1 / 6.2; 8 lanes, 20000 x 17 35 / 15, 1500 x 128
// 8.7 / 8.9, 500 x 128 7.1 / 8.1; 16 lanes, 20000 x 17 37 / 18, 4000 x 200 35 / 21, 1500 x 128 10.8 / 12.8, 3000 x 30 and 5 x 10000
// 11.5 / 16.1.
constexpr int kWaveLanesLog2 = 4;
inline bool long_rows_by_wave(int pieces, int lanes_log2) {
  return lanes_log2 <= kWaveLanesLog2 && pieces > (lanes_log2 <= 2 ? 1024 : 256 << lanes_log2);
}
__host__ __device__ inline int long_blocks(int pieces, bool by_wave) { return by_wave ? (pieces + 3) / 4 : pieces; }

// 1 where a block's piece is half a chunk: where rows are wide, a block's groups are few and its share of 128 entries is the
// longest chain of a launch that leaves the chip idle.  A layer's backward with 1500 destinations, us, with pieces of 16 entries
// and a launch of its own for their sums / whole chunks / halves: one row of 180 entries, 512 features in fp32 25.0 / 30.5 / 24.2,
// 1024 in bf16 25.4 / 32.4 / 25.0; 300 rows of 128 entries, 1024 in bf16 30.8 / 29.6 / 32.7.
inline int long_halves(int chunks, int lanes_log2) { return lanes_log2 > kWaveLanesLog2 && chunks <= kHalvedChunks ? 1 : 0; }

// The piece of the calling thread: the block's, or its wavefront's.  `on`: whether there is one (the wavefronts behind the last
// piece stand in for it up to the barrier).  Threads first, first + step, ... bring its entries to its part of an LDS array.
template <bool WAVE> struct LongSlot {
  int item, lds, first, step;
  bool on;
  __device__ __forceinline__ explicit LongSlot(int pieces) {
    const int w = threadIdx.x >> 6;
    item = WAVE ? (int)blockIdx.x * 4 + w : (int)blockIdx.x;
    on = item < pieces;
    item = min(item, pieces - 1);
    lds = WAVE ? w * kChunk : 0;
    first = WAVE ? threadIdx.x & 63 : threadIdx.x;
    step = WAVE ? 64 : 256;
  }
};

template <int N> struct LongLds {   // of a block that takes one piece
  float red[4 * 64 * N];
  uint32_t before;   // blocks of the row that finished before this one
};

// One vector of a piece's partial sum, past the L2 (device scope).
template <int N> __device__ __forceinline__ void put_partial(float *at, const float (&acc)[N]) {
  unsigned long long *o = reinterpret_cast<unsigned long long *>(at);
#pragma unroll
  for (int k = 0; k < N; k += 2)
    __hip_atomic_store(o + k / 2, (unsigned long long)__float_as_uint(acc[k]) | ((unsigned long long)__float_as_uint(acc[k + 1]) << 32),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Adds the same vector of the partial sums g, g + groups, ... of n, `pitch` floats apart.  A source of 50k destinations has 400 of
// them, so U are in flight as long as there are U: 16 floats a lane where a block takes a piece, which leaves the launch's short
// rows their eight wavefronts per SIMD, 32 where a wavefront does.
template <int N, int U> __device__ __forceinline__ void add_partials(float (&acc)[N], const float *at, int pitch, int g, int groups, int n) {
  auto take = [&](auto count, int j) {
    constexpr int C = decltype(count)::value;
    unsigned long long v[C][N / 2];
#pragma unroll
    for (int u = 0; u < C; ++u) {
      const unsigned long long *o = reinterpret_cast<const unsigned long long *>(at + (int64_t)(j + u * groups) * pitch);
#pragma unroll
      for (int k = 0; k < N / 2; ++k) v[u][k] = __hip_atomic_load(o + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int u = 0; u < C; ++u)
#pragma unroll
      for (int k = 0; k < N; k += 2) {
        acc[k] += __uint_as_float((uint32_t)v[u][k / 2]);
        acc[k + 1] += __uint_as_float((uint32_t)(v[u][k / 2] >> 32));
      }
  };
  int j = g;
  for (; j + (U - 1) * groups < n; j += U * groups) take(std::integral_constant<int, U>{}, j);
  for (; j < n; j += groups) take(std::integral_constant<int, 1>{}, j);
}
// Called by the wavefront that stored a piece's partial sum: its stores are at the coherence point before the count goes up.
// Returns how many pieces of the row were there before.
__device__ __forceinline__ uint32_t count_piece(uint32_t *count) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  uint32_t before = 0;
  if ((threadIdx.x & 63) == 0) before = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  before = __shfl(before, 0);
  asm volatile("" ::: "memory");   // no load of a partial sum in front of it
  return before;
}

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
      put_partial<N>(partial + (int64_t)item * pitch + q * N, acc);
    }
  }
  if (p.pieces == 1) return;
  if (wave == 0) {   // the one that stored
    const uint32_t before = count_piece(count + p.row);
    if (lane == 0) sm.before = before;
  }
  __syncthreads();
  if (sm.before != (uint32_t)(p.pieces - 1)) return;
  for (int q0 = 0; q0 < nvec; q0 += lanes) {
    const int q = q0 + col;
    float acc[N];
#pragma unroll
    for (int k = 0; k < N; ++k) acc[k] = 0.f;
    if (q < nvec) add_partials<N, 16 / N>(acc, partial + (int64_t)p.first * pitch + q * N, pitch, g, groups, p.pieces);
    if (meet(acc) && q < nvec) done(q, acc);
  }
}

// The same by one wavefront, for rows of at most 2^l2 <= 16 vectors; no barrier.
template <int N, typename Sum, typename Done>
__device__ __forceinline__ void long_row_wave(const LongPiece &p, int item, int l2, int nvec, float *partial, int pitch, uint32_t *count,
                                              Sum sum, Done done) {
  const int lane = threadIdx.x & 63, lanes = 1 << l2, groups = 64 >> l2, q = lane & (lanes - 1), g = lane >> l2;
  float acc[N];
  auto clear = [&]() {
#pragma unroll
    for (int k = 0; k < N; ++k) acc[k] = 0.f;
  };
  auto meet = [&]() {   // every lane gets its vector's sum over the groups
    for (int o = lanes; o < 64; o <<= 1) {
#pragma unroll
      for (int k = 0; k < N; ++k) acc[k] += __shfl_xor(acc[k], o);
    }
  };
  clear();
  if (q < nvec) sum(q, g, groups, acc);
  meet();
  const bool mine = lane < lanes && q < nvec;
  if (p.pieces == 1) {
    if (mine) done(q, acc);
    return;
  }
  if (mine) put_partial<N>(partial + (int64_t)item * pitch + q * N, acc);
  if (count_piece(count + p.row) != (uint32_t)(p.pieces - 1)) return;
  clear();
  if (q < nvec) add_partials<N, 32 / N>(acc, partial + (int64_t)p.first * pitch + q * N, pitch, g, groups, p.pieces);
  meet();
  if (mine) done(q, acc);
}

template <bool WAVE, int N, typename Sum, typename Done>
__device__ __forceinline__ void long_row(const LongPiece &p, int item, int l2, int nvec, LongLds<N> &sm, float *partial, int pitch,
                                         uint32_t *count, Sum sum, Done done) {
  if constexpr (WAVE) long_row_wave<N>(p, item, l2, nvec, partial, pitch, count, sum, done);
  else long_row_piece<N>(p, item, l2, nvec, sm, partial, pitch, count, sum, done);
}

}  // namespace hgnn
