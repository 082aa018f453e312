// Block reductions, the loss-mask count and the token walk shared by the per-token
// kernels. Every reduction here runs in a fixed order, so results do not depend on
// scheduling.
#pragma once

#include "common.hpp"

namespace sao {

// Sum over a block of THREADS threads (a multiple of 64); every thread gets the
// result. `sh` holds THREADS / 64 elements.
template <int THREADS, typename T>
__device__ __forceinline__ T block_sum(T v, T* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  T r = sh[0];
#pragma unroll
  for (int w = 1; w < THREADS / 64; ++w) r += sh[w];
  return r;
}

// N sums over the block at once, left in thread 0: the lane moves of the N values
// overlap and one barrier serves them all. (Seven calls of block_sum in a row took
// about half of an 11 us loss pass over 65,536 tokens.) `sh` holds THREADS / 64 rows.
template <int THREADS, int N, typename T>
__device__ __forceinline__ void block_sums(T (&v)[N], T (*sh)[N]) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < N; ++i) sh[wave][i] = v[i];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int i = 0; i < N; ++i) {
      v[i] = sh[0][i];
#pragma unroll
      for (int w = 1; w < THREADS / 64; ++w) v[i] += sh[w][i];
    }
}

// Per-block partial sums of the mask (grid-stride).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_mask_count(const uint8_t* mask, int64_t T, int64_t* part) {
  __shared__ int64_t sh[THREADS / 64];
  int64_t c = 0;
  const bool vec = (reinterpret_cast<uintptr_t>(mask) & 7u) == 0;
  const int64_t words = vec ? T / 8 : 0;
  const int64_t step = static_cast<int64_t>(gridDim.x) * THREADS;
  const int64_t first = static_cast<int64_t>(blockIdx.x) * THREADS + threadIdx.x;
  for (int64_t i = first; i < words; i += step) {
    const uint64_t x = reinterpret_cast<const uint64_t*>(mask)[i];
    // The top bit of each byte that is not zero.
    constexpr uint64_t k7f = 0x7f7f7f7f7f7f7f7full;
    c += __popcll((((x & k7f) + k7f) | x) & ~k7f);
  }
  for (int64_t t = 8 * words + first; t < T; t += step) c += mask[t] != 0 ? 1 : 0;
  c = block_sum<THREADS>(c, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = c;
}

// The loss-mask count that a pass divides by: the caller's, or the sum of the
// k_mask_count partials of this call, which every block adds up for itself (a launch
// of their own for at most 256 of them, in the critic 1024, would cost more). The
// partials are not the workspace's other pieces, which the blocks write.
struct TokenCount {
  const int64_t* n;     // or null
  const int64_t* part;
  int blocks;
  template <int THREADS>
  __device__ __forceinline__ int64_t get() const {
    if (n) return *n;
    __shared__ int64_t sh[THREADS / 64];
    int64_t c = 0;
    for (int i = threadIdx.x; i < blocks; i += THREADS) c += part[i];
    return block_sum<THREADS>(c, sh);
  }
};

// Token walk of the per-token kernels. Each wave takes chunks of 256 or 512 (QUADS 1 or
// 2) consecutive tokens (grid-stride over chunks); lane l handles tokens 4l .. 4l+3,
// and 256 + 4l .. 256 + 4l+3, of a chunk, so every load and store instruction of a
// whole chunk covers one contiguous span. quad(t) handles tokens t .. t+3 with
// 16-byte vector access (whole chunks, when vec_ok); one(t) handles a single
// token (the ragged tail, or every token when the bases do not allow vectors).
template <int THREADS, int QUADS, class Quad, class One>
__device__ __forceinline__ void walk_tokens(int64_t T, bool vec_ok, Quad&& quad, One&& one) {
  constexpr int kWalkChunk = 256 * QUADS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t waves = static_cast<int64_t>(gridDim.x) * (THREADS / 64);
  for (int64_t w0 = (static_cast<int64_t>(blockIdx.x) * (THREADS / 64) + wave) * kWalkChunk; w0 < T;
       w0 += waves * kWalkChunk) {
    if (vec_ok && w0 + kWalkChunk <= T) {
#pragma unroll
      for (int q = 0; q < QUADS; ++q) quad(w0 + 256 * q + 4 * lane);
    } else {
      for (int j = 0; j < 4 * QUADS; ++j) {
        const int64_t t = w0 + 256 * (j / 4) + 4 * lane + j % 4;
        if (t < T) one(t);
      }
    }
  }
}

}  // namespace sao
