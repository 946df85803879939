// Output stage shared by the list builders: one wave (emit_row_wave) or one
// workgroup of 256 lanes (emit_row) writes the list row of one (b, h, query
// tile) from a keep predicate over logical key tiles 0 .. nk_cap-1 (false at
// and beyond nk).  A wave ballot gives two 32-bit mask words; the kept indices
// are placed in ascending order, and the tail of the row is padded with -1.
// A wave per row needs no barrier (four rows run side by side in a workgroup);
// a workgroup per row takes 256 tiles per pass with two barriers, and is for few
// or long rows (list_rule.h) and top-k rows of more than 2,048 candidates.
#pragma once

#include "../launch.h"

namespace uf {
namespace lists {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

template <class Keep>
__device__ void emit_row_wave(Keep keep_of, int nk_cap, int mask_words, int32_t* count, int32_t* idx, uint32_t* mask) {
  const int lane = threadIdx.x & 63;
  int base = 0;
  for (int j0 = 0; j0 < nk_cap; j0 += 256) {
    bool keep[4];                            // four words decided side by side
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = j0 + 64 * k + lane;
      keep[k] = (j < nk_cap) && keep_of(j);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t ballot = __ballot(keep[k]);
      const int w0 = (j0 + 64 * k) >> 5;
      if (lane < 2 && w0 + lane < mask_words) mask[w0 + lane] = uint32_t(ballot >> (32 * lane));
      if (keep[k]) idx[base + __popcll(ballot & ((1ull << lane) - 1ull))] = j0 + 64 * k + lane;
      base += __popcll(ballot);
    }
  }
  for (int j = base + lane; j < nk_cap; j += 64) idx[j] = -1;
  if (lane == 0) *count = base;
}

// `wave_count` is a __shared__ int[kWaves] of the calling kernel.  Every lane
// of the workgroup must call this (it contains barriers).
template <class Keep>
__device__ void emit_row(Keep keep_of, int nk_cap, int mask_words, int32_t* count, int32_t* idx,
                         uint32_t* mask, int* wave_count) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int base = 0;
  for (int j0 = 0; j0 < nk_cap; j0 += kThreads) {
    const int j = j0 + threadIdx.x;
    const bool keep = (j < nk_cap) && keep_of(j);
    const uint64_t ballot = __ballot(keep);
    const int w0 = (j0 + wave * 64) >> 5;
    if (lane == 0 && w0 < mask_words) mask[w0] = uint32_t(ballot);
    if (lane == 0 && w0 + 1 < mask_words) mask[w0 + 1] = uint32_t(ballot >> 32);
    if (lane == 0) wave_count[wave] = __popcll(ballot);
    __syncthreads();
    int off = base, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      off += (w < wave) ? wave_count[w] : 0;
      total += wave_count[w];
    }
    if (keep) idx[off + __popcll(ballot & ((1ull << lane) - 1ull))] = j;
    __syncthreads();
    base += total;
  }
  for (int j = base + threadIdx.x; j < nk_cap; j += kThreads) idx[j] = -1;
  if (threadIdx.x == 0) *count = base;
}

}  // namespace lists
}  // namespace uf
