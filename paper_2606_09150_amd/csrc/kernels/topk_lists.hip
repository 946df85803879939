// topk_lists: per (b, h, query tile) keep lists by content-adaptive top-k.
//
// Realises the content-adaptive selection of Sec. 2.3.1 (b), Eq. 4: queries
// and keys are mean-pooled per tile, each (query tile, key tile) pair gets the
// dot product of the pooled vectors as its score, and every query tile keeps
// the `budget` best-scoring key tiles among the ranked candidates (the softmax
// and 1/sqrt(d) of Eq. 4 are monotone and do not change the ranking).  Tiles
// of the pinned and of the current chunk are kept without ranking when the
// rule asks for it; the lists are intersected with the temporal causal mask
// by construction (only the window's tiles exist).
//
// Arithmetic is IEEE float32 in a fixed order, so that the integer decision is
// reproducible: a pooled query is the sequential sum of the tile's valid rows
// divided once by their count (pooled keys come from the append kernel in the
// same form); a score adds the rounded products in order of d, with fused
// multiply-add disabled; scores compare through the unsigned key that orders
// float32 like the real line, equal keys going to the lower tile index.
//
// Three kernels.  pool_queries: one workgroup per query tile stages the tile's
// valid rows in LDS and lane d adds column d in token order, writing the
// pooled query into the list buffer's scratch section.  topk_scores: one
// workgroup per head, 32 query tiles and 32 ranked candidates, both sides'
// pooled vectors in LDS, two by two scores per lane (four independent chains);
// the order keys go to the row's index section, which is at least as long and is
// rewritten last.  topk_select: one wave per row (four waves for the longest
// rows) holds the row's keys in registers and finds the budget-th largest one
// bit by bit, from ballots: the largest T with at least `budget` keys >= T, ending
// as soon as the count is exact.  Every larger key is kept, then the first equal
// ones (ties to the lower index), and the wave writes its row.
//
// What bounds them: pool_queries reads Q (75 MB at 1K, 14.4 us, 5.2 TB/s, the
// rate of a large copy; 17.8 us with a loop that had one load per lane in flight,
// the lists 47.2 -> 42.4 us); the scores are
// 2 x 128 unfused operations per pair (about 9 us of vector issue at 1K, 2,304
// rows by 576 candidates); the selection is latency.  One kernel that scored two
// query tiles against every candidate read each pooled key once per two rows (340
// MB from L2) and selected with histograms in two of its four waves: 66 us for
// what topk_scores and topk_select now do in 15 + 13 us.  Windows with few
// rows and candidates take two kernels: topk_select computes its row's keys.
// (That form was slower than the one kernel where rows were few, as a workgroup held
// four rows and a wave all candidates of one, eight chunks of their keys in flight:
// 8 rows x 124 candidates 15.3 us in one kernel, then 18.5, and 14.5 with a workgroup
// per row and a wave per 64 candidates.)
#include "../list_rule.h"
#include "list_emit.h"

#pragma clang fp contract(off)

namespace uf {
namespace {

using lists::kThreads;
using lists::kWaves;
constexpr int kD = 128;

__device__ inline float bf16_to_f32(uint16_t x) { return __uint_as_float(uint32_t(x) << 16); }

// Unsigned key that orders float32 values like the real line.
__device__ inline uint32_t order_key(float s) {
  const uint32_t u = __float_as_uint(s);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <int T>
__global__ __launch_bounds__(kThreads) void pool_queries_kernel(TopkArgs a) {
  constexpr int kChunks = kD / 8;        // 16-byte chunks of a row
  constexpr int kPer = T * kChunks / kThreads, kStep = kThreads / kChunks;
  __shared__ uint4 stage[T * kChunks];
  const int row = blockIdx.x;            // (b*H + h)*NT + i
  const int i = row % a.NT;
  const int bh = row / a.NT;
  const int h = bh % a.H;
  const int b = bh / a.H;
  const int nv = tile_valid(a.tv, i, a.NT, a.tail, T);
  // every load of the thread before any store to LDS; rows past the last valid
  // one repeat it (and are not summed), so that no load has a branch
  const int r0 = threadIdx.x / kChunks, cc = threadIdx.x % kChunks;
  uint4 chunk[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    chunk[k] = *reinterpret_cast<const uint4*>(
        a.q + ((size_t(b) * a.L + size_t(i) * T + min(r0 + kStep * k, nv - 1)) * a.H + h) * kD + cc * 8);
#pragma unroll
  for (int k = 0; k < kPer; ++k) stage[(r0 + kStep * k) * kChunks + cc] = chunk[k];
  __syncthreads();
  if (threadIdx.x < kD) {
    const uint16_t* st = reinterpret_cast<const uint16_t*>(stage);
    const int d = threadIdx.x;
    float acc = 0.f;
#pragma unroll 8
    for (int r = 0; r < nv; ++r) acc += bf16_to_f32(st[r * kD + d]);
    float* qmean = reinterpret_cast<float*>(a.lists + a.scratch_offset);
    qmean[size_t(row) * kD + d] = acc / float(nv);
  }
}

constexpr int kTile = 32;                 // query tiles and candidates of a workgroup
constexpr int kRow = kD + 4;              // LDS row in floats: 16 rows' chunks cover all banks

__global__ __launch_bounds__(kThreads) void topk_scores_kernel(TopkArgs a) {
  __shared__ float4 sq[kTile * kRow / 4], sk[kTile * kRow / 4];
  const int nc = a.cand_hi - a.cand_lo;    // ranked candidates of a row
  const unsigned mt = unsigned(nc + kTile - 1) / kTile, it = unsigned(a.NT + kTile - 1) / kTile;
  const int m0 = int(blockIdx.x % mt) * kTile, i0 = int(blockIdx.x / mt % it) * kTile, bh = int(blockIdx.x / mt / it);
  const float4* qmean = reinterpret_cast<const float4*>(a.lists + a.scratch_offset);
  const size_t slot_pages = size_t(a.B) * a.H * a.NT;
  // 32 rows of 32 chunks each, two rows per wave and pass (so that a row's slot is
  // a scalar load of the kernel arguments); rows past the end repeat the last
  // one, and are not written
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool odd = (threadIdx.x & 32) != 0;
  const int cc = threadIdx.x & 31;
  auto pooled = [&](int r) {
    const int j = a.cand_lo + min(m0 + r, nc - 1);
    const int pos = j / a.NT;
    return reinterpret_cast<const float4*>(a.kmean) +
           (size_t(a.slot_of[pos]) * slot_pages + size_t(bh) * a.NT + (j - pos * a.NT)) * (kD / 4);
  };
#pragma unroll
  for (int k = 0; k < kTile / 8; ++k) {
    const int ra = 8 * k + 2 * wave, r = odd ? ra + 1 : ra;
    const float4* pa = pooled(ra);
    const float4* pb = pooled(ra + 1);
    sq[r * (kRow / 4) + cc] = qmean[(size_t(bh) * a.NT + min(i0 + r, a.NT - 1)) * (kD / 4) + cc];
    sk[r * (kRow / 4) + cc] = (odd ? pb : pa)[cc];
  }
  __syncthreads();
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;   // candidates tx, tx + 16; rows ty, ty + 16
  float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll 8
  for (int c = 0; c < kD / 4; ++c) {
    float4 q[2], k[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      q[u] = sq[(ty + 16 * u) * (kRow / 4) + c];
      k[u] = sk[(tx + 16 * u) * (kRow / 4) + c];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        acc[u][v] = acc[u][v] + q[u].x * k[v].x;
        acc[u][v] = acc[u][v] + q[u].y * k[v].y;
        acc[u][v] = acc[u][v] + q[u].z * k[v].z;
        acc[u][v] = acc[u][v] + q[u].w * k[v].w;
      }
  }
  uint32_t* keys = reinterpret_cast<uint32_t*>(a.lists + a.idx_offset);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int i = i0 + ty + 16 * u, m = m0 + tx + 16 * v;
      if (i < a.NT && m < nc) keys[(size_t(bh) * a.NT + i) * a.nk_cap + m] = order_key(acc[u][v]);
    }
}

// W waves per row, K keys per lane (64 W K >= candidates).  RANK: the budget
// cuts the candidates (otherwise all of them are kept, or none).  SCORE: the
// row's waves compute its keys themselves (a lane takes a candidate) instead of
// reading those of topk_scores; ALONE: each row in a workgroup of its own, so
// that few rows spread over as many CUs, and a lane requests its candidate's
// whole pooled key (512 bytes) before it uses any of it.
enum Keys { kRead, kScore, kScoreAlone };
template <int W, int K, bool RANK, Keys KEYS>
__global__ __launch_bounds__(KEYS == kScoreAlone ? 64 * W : kThreads) void topk_select_kernel(TopkArgs a) {
  constexpr bool SCORE = KEYS != kRead, ALONE = KEYS == kScoreAlone;
  static_assert(!SCORE || (RANK && (ALONE ? K == 1 : W == 1)), "rows scored in place");
  constexpr int kRows = ALONE ? 1 : kWaves / W;   // rows of a workgroup
  constexpr int kWords = W * K;            // 64-candidate words of a row
  __shared__ uint64_t sgt[RANK ? kRows : 1][RANK ? kWords : 1], seq[RANK ? kRows : 1][RANK ? kWords : 1];
  __shared__ int part[2][kWaves];
  const int nc = max(a.cand_hi - a.cand_lo, 0);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = wave % W, slot = wave / W;
  const int row = blockIdx.x * kRows + slot;
  if (row >= a.B * a.H * a.NT) return;     // W = 1 only: whole waves, and no barrier follows
  int32_t* idx = reinterpret_cast<int32_t*>(a.lists + a.idx_offset) + size_t(row) * a.nk_cap;

  if constexpr (RANK) {
    // candidate 64 (sub + W i) + lane; a key of 0 past the end is below every trial value
    uint32_t key[K];
    if constexpr (SCORE) {
      __shared__ float4 sqm[kRows][kD / 4];
      const int bh = row / a.NT;
      if (lane < kD / 4)                     // (every wave of the row writes the same)
        sqm[slot][lane] = reinterpret_cast<const float4*>(a.lists + a.scratch_offset)[size_t(row) * (kD / 4) + lane];
      if constexpr (W > 1) __syncthreads();
      else __builtin_amdgcn_wave_barrier();
      const float4* kp[K];
      float acc[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int j = a.cand_lo + min(64 * (sub + W * i) + lane, nc - 1);
        const int pos = j / a.NT;
        kp[i] = reinterpret_cast<const float4*>(a.kmean) +
                (size_t(a.slot_of[pos]) * a.B * a.H * a.NT + size_t(bh) * a.NT + (j - pos * a.NT)) * (kD / 4);
        acc[i] = 0.f;
      }
      constexpr int kAhead = ALONE ? kD / 4 : 8;   // chunks requested at a time
#pragma unroll 1
      for (int c0 = 0; c0 < kD / 4; c0 += kAhead) {
        float4 k[K][kAhead];
#pragma unroll
        for (int c = 0; c < kAhead; ++c)
#pragma unroll
          for (int i = 0; i < K; ++i) k[i][c] = kp[i][c0 + c];
#pragma unroll
        for (int c = 0; c < kAhead; ++c) {
          const float4 q = sqm[slot][c0 + c];
#pragma unroll
          for (int i = 0; i < K; ++i) {
            acc[i] = acc[i] + q.x * k[i][c].x;
            acc[i] = acc[i] + q.y * k[i][c].y;
            acc[i] = acc[i] + q.z * k[i][c].z;
            acc[i] = acc[i] + q.w * k[i][c].w;
          }
        }
      }
#pragma unroll
      for (int i = 0; i < K; ++i) key[i] = 64 * (sub + W * i) + lane < nc ? order_key(acc[i]) : 0u;
    } else {
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int m = 64 * (sub + W * i) + lane;
        key[i] = m < nc ? uint32_t(idx[m]) : 0u;
      }
    }
    int flip = 0;
    auto total = [&](int c) {              // over the row's waves
      if constexpr (W > 1) {
        if (lane == 0) part[flip][wave] = c;
        __syncthreads();
        c = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) c += part[flip][w];
        flip ^= 1;
      }
      return __builtin_amdgcn_readfirstlane(c);
    };
    uint32_t T = 0;
    bool exact = false;
    for (int bit = 31; bit >= 0 && !exact; --bit) {
      const uint32_t t = T | (1u << bit);
      int c = 0;
#pragma unroll
      for (int i = 0; i < K; ++i) c += __popcll(__ballot(key[i] >= t));
      c = total(c);
      if (c >= a.budget) T = t;
      exact = c == a.budget;
    }
    // the keys above T (exact: and T itself, on which the count ended)
    int above = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const int m = 64 * (sub + W * i) + lane;
      const uint64_t gt = __ballot(exact ? key[i] >= T : key[i] > T);
      const uint64_t eq = __ballot(!exact && m < nc && key[i] == T);
      above += __popcll(gt);
      if (lane == 0) {
        sgt[slot][sub + W * i] = gt;
        seq[slot][sub + W * i] = eq;
      }
    }
    const int need = a.budget - total(above);   // equal keys still admitted, in index order
    if constexpr (W > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();
    if (sub == 0) {
      constexpr int kPer = (kWords + 63) / 64;
      int before = 0;
      uint64_t w[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int n = lane * kPer + u;
        w[u] = n < kWords ? seq[slot][n] : 0;
        before += __popcll(w[u]);
      }
      const int own = before;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(before, o);
        if (lane >= o) before += y;
      }
      int left = need - (before - own);
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int n = lane * kPer + u;
        uint64_t take = 0, rest = w[u];
        const int equal = int(__popcll(rest));   // (the builtin's type is unsigned)
        if (left >= equal) take = rest;
        else
          for (int e = 0; e < left; ++e) {       // the lowest `left` bits
            take |= rest & -rest;
            rest &= rest - 1;
          }
        left -= equal;
        if (n < kWords) sgt[slot][n] |= take;
      }
    }
    if constexpr (W > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();
  }

  if (ALONE && sub != 0) return;           // the first wave writes the row; no barrier follows
  const int qi = row % a.NT;
  auto keep_of = [&](int j) {
    if (j >= a.nk) return false;
    if (!tile_local(a.tv, qi, j % a.NT)) return false;   // structural local window (block geometry)
    if (j < a.cand_lo || j >= a.cand_hi) return true;    // forced: pinned or current chunk
    if constexpr (!RANK) return a.budget > 0;
    const int m = j - a.cand_lo;
    return ((sgt[slot][m >> 6] >> (m & 63)) & 1u) != 0;
  };
  int32_t* count = reinterpret_cast<int32_t*>(a.lists) + row;
  uint32_t* mask = reinterpret_cast<uint32_t*>(a.lists + a.mask_offset) + size_t(row) * a.mask_words;
  if constexpr (W == 1 || ALONE)
    lists::emit_row_wave(keep_of, a.nk_cap, a.mask_words, count, idx, mask);
  else
    lists::emit_row(keep_of, a.nk_cap, a.mask_words, count, idx, mask, part[0]);
}

}  // namespace

hipError_t launch_topk_lists(const TopkArgs& a, hipStream_t stream) {
  const unsigned rows = unsigned(a.B) * unsigned(a.H) * unsigned(a.NT);
  const int nc = a.cand_hi > a.cand_lo ? a.cand_hi - a.cand_lo : 0;
  hipError_t e = hipSuccess;
  // a budget of none or of every candidate needs no score
  if (a.budget == 0 || a.budget >= nc) {
    topk_select_kernel<1, 1, false, kRead><<<(rows + 3) / 4, kThreads, 0, stream>>>(a);
    return hipGetLastError();
  }
  if (a.T == 128)
    pool_queries_kernel<128><<<rows, kThreads, 0, stream>>>(a);
  else
    pool_queries_kernel<64><<<rows, kThreads, 0, stream>>>(a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const unsigned four = (rows + 3) / 4;
  // Few pairs: a launch costs more than reading each pooled key once per row.
  const unsigned waves = unsigned(nc + 63) / 64;
  if (topk_row_alone(int(rows), nc)) {
    if (waves == 1) topk_select_kernel<1, 1, true, kScoreAlone><<<rows, 64, 0, stream>>>(a);
    else if (waves == 2) topk_select_kernel<2, 1, true, kScoreAlone><<<rows, 128, 0, stream>>>(a);
    else topk_select_kernel<4, 1, true, kScoreAlone><<<rows, 256, 0, stream>>>(a);
    return hipGetLastError();
  }
  // More rows of few candidates, four to a workgroup; two launches against three:
  // 1,500 rows x 50 21.6 against 23.1 us, 4,000 x 20 34.7 against 36.1, 640 x 120
  // 16.4 against 16.7; 960 x 120 18.5 either way, 2,560 x 64 28.5 either way.
  if (waves <= 2 && uint64_t(rows) * uint64_t(nc) <= 80000) {
    if (waves == 1) topk_select_kernel<1, 1, true, kScore><<<four, kThreads, 0, stream>>>(a);
    else topk_select_kernel<1, 2, true, kScore><<<four, kThreads, 0, stream>>>(a);
    return hipGetLastError();
  }
  const unsigned tiles = (unsigned(a.NT + kTile - 1) / kTile) * (unsigned(nc + kTile - 1) / kTile);
  topk_scores_kernel<<<tiles * unsigned(a.B) * unsigned(a.H), kThreads, 0, stream>>>(a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // Keys per lane: every one that a row does not need costs 0.2 to 0.8 us (2,304 rows
  // of 384: 6 keys 35.9 us, 8 36.4, 10 37.2, 16 39.3; of 576: 10 42.3, 12 42.8, 16 44.5; 444
  // of 222: 4 18.1, 10 21.1), so a few steps; 10 serves 257 to 640 candidates.  32 keys
  // spill 53 scalar registers (the ballots) and are still the better form of many rows:
  // 3,000 rows of 1,500 86 us, four waves of 8 keys 92, of 16 keys 105 (500 rows: 42, 31 and 34).
  // Past 2,048 a row takes four waves: against one of 64 keys, which spill 207, 250 rows of
  // 3,000 32.5 and 64.8 us, 1,000 of 4,000 71 and 96, 3,000 of 3,000 141 and 147.  Four waves of
  // 64 keys take 61 us for 250 rows of 4,000 and 122 for 1,000, and are for the rest.
  if (nc <= 64 * 4) topk_select_kernel<1, 4, true, kRead><<<four, kThreads, 0, stream>>>(a);
  else if (nc <= 64 * 10) topk_select_kernel<1, 10, true, kRead><<<four, kThreads, 0, stream>>>(a);
  else if (nc <= 64 * 16) topk_select_kernel<1, 16, true, kRead><<<four, kThreads, 0, stream>>>(a);
  else if (nc <= 64 * 32) topk_select_kernel<1, 32, true, kRead><<<four, kThreads, 0, stream>>>(a);
  else if (nc <= 64 * 64) topk_select_kernel<4, 16, true, kRead><<<rows, kThreads, 0, stream>>>(a);
  else topk_select_kernel<4, 64, true, kRead><<<rows, kThreads, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace uf
