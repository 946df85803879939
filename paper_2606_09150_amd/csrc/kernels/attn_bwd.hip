// attn_bwd: gradients of the block-sparse chunk-causal attention.
//
// The student of Phase I is trained through the sparse causal attention of
// Sec. 2.3.1 (the Eq. 4 mask inside the generator that the DMD objective
// updates), so the training side needs dQ, dK and dV over the same keep
// lists.  With p = exp(scale*q.k - lse) over the kept keys of a row,
// delta = <dO, O>, dS = P (dO V^T - delta):
//   dV = P^T dO,  dK = scale dS^T Q,  dQ = scale dS K.
//
// Three kernels, all with 32x32x16 bf16 MFMA and fp32 accumulation, each a
// template on the tile size T (128 or 64; the wave counts below are for 128
// and halve for 64):
//  * prep: per query tile, Q and dO rows (rows past the chunk end zero),
//    -LSE/scale (-inf on those rows, so that their weights vanish) and
//    -delta, which seed the S and dP accumulators;
//  * dkdv: one workgroup of eight waves per window key tile (one per CU).
//    Waves w and w + 4 share 32 keys.  The workgroup gathers the query tiles
//    whose mask bit keeps its tile and walks them in half tiles: wave w
//    computes S = Q K^T and P, hands P to wave w + 4 through LDS and accumulates
//    dV^T += dO^T P, while wave w + 4 computes dP = dO V^T, dS = P (dP - delta)
//    from the shared P and accumulates dK^T += Q^T dS one half tile later; Q and
//    dO rows are copied two half tiles ahead;
//  * dq: one workgroup of four waves per query tile (two per CU; four waves with
//    either tile size), 32 queries per wave; it walks the row's list in units of
//    64 keys and per 32-key block computes S^T = K Q^T, dP^T = V dO^T, dS^T, then
//    dQ^T += K^T dS^T, while the next unit is copied;
// The transposed operands (dO^T, Q^T, K^T, and V rows from the pool's V^T)
// come from row-major LDS tiles through the transposing LDS read
// (ds_read_b64_tr_b16), so each tile is copied into LDS once, in the layout the
// pool or the workspace already holds.  No atomics: every output row is owned
// by one workgroup, so results are reproducible.
#include <mutex>
#include <type_traits>

#include "attn_common.h"
#include "../launch_bwd.h"

namespace uf {
namespace {

using namespace attn;

constexpr int kT = 128;
constexpr int kThreads = 256;                  // four waves
constexpr uint32_t kTile = 32768;              // one [128][128] bf16 tile

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;
typedef __attribute__((address_space(3))) uint8_t lds_u8;

__device__ inline float bf16f(uint16_t x) { return __uint_as_float(uint32_t(x) << 16); }

// ---------------------------------------------------------------- prep ----

// T-token tiles; a record always has room for 128 rows and 128 per-query
// values, of which the first T are used.  HBM-bound: Q, dO and O are read once and
// a record written; 16 lanes hold a row's chunks, so delta = <dO, O> is formed
// from the chunks of the copy and added over them.  1K window (2,304 records, 377
// MB): 123 -> 63 us, 6 TB/s (one lane per query that read its O and dO rows
// again, two bytes at a time, before).
template <int T>
__global__ __launch_bounds__(kThreads) void bwd_prep_kernel(BwdArgs a) {
  const int row = blockIdx.x;                  // (b*H + h)*NT + i
  const int i = row % a.NT;
  const int bh = row / a.NT;
  const int h = bh % a.H, b = bh / a.H;
  const int nv = tile_valid(a.tv, i, a.NT, a.tail, T);
  uint8_t* rec = a.work + size_t(row) * kBwdQTile;
  float* nlse = reinterpret_cast<float*>(rec + 2 * kTile);
  float* ndelta = nlse + kT;
  constexpr int kPer = T * 16 / kThreads;      // 16-byte chunks of a thread, kThreads/16 rows apart
  const int cc = threadIdx.x & 15, r0 = threadIdx.x >> 4;
  uint4 vq[kPer], vg[kPer], vo[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {             // every load before the first store
    const int r = r0 + k * (kThreads / 16);
    vq[k] = vg[k] = vo[k] = make_uint4(0, 0, 0, 0);
    if (r < nv) {
      const size_t off = ((size_t(b) * a.L + size_t(i) * T + r) * a.H + h) * kD + cc * 8;
      vq[k] = *reinterpret_cast<const uint4*>(a.q + off);
      vg[k] = *reinterpret_cast<const uint4*>(a.dout + off);
      vo[k] = *reinterpret_cast<const uint4*>(a.o + off);
    }
  }
  float nl = -INFINITY;
  if (threadIdx.x < T && int(threadIdx.x) < nv)
    nl = -a.lse[(size_t(b) * a.H + h) * a.L + size_t(i) * T + threadIdx.x] / a.scale;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = r0 + k * (kThreads / 16), c = r * 16 + cc;
    reinterpret_cast<uint4*>(rec)[c] = vq[k];
    reinterpret_cast<uint4*>(rec + kTile)[c] = vg[k];
    const uint32_t g[4] = {vg[k].x, vg[k].y, vg[k].z, vg[k].w}, o[4] = {vo[k].x, vo[k].y, vo[k].z, vo[k].w};
    float dl = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      dl += bf16f(uint16_t(o[e])) * bf16f(uint16_t(g[e])) + bf16f(uint16_t(o[e] >> 16)) * bf16f(uint16_t(g[e] >> 16));
#pragma unroll
    for (int s = 1; s < 16; s <<= 1) dl += __shfl_xor(dl, s, 16);
    if (cc == 0) ndelta[r] = -dl;
  }
  if (threadIdx.x < T) nlse[threadIdx.x] = nl;
}

// ------------------------------------------------------------- shared ----

// LDS layout of a [128][128] bf16 tile: 16-byte chunk c of row r sits at
// position perm(c) ^ f(r) of the row, perm swapping bits 1 and 3 of c and
// f(r) = (r3, r1, r0, r2 ^ r3) (bits 3..0).  Both 16-byte row reads (eight or
// sixteen consecutive rows, or rows in swap23 order, one chunk) and the
// transposing 8-byte reads (four consecutive rows, four consecutive chunks
// per 32 lanes) then touch every bank once per cycle, with 32 or 64 banks.
__device__ inline int swz_perm(int c) { return (c & ~10) | ((c & 2) << 2) | ((c & 8) >> 2); }
__device__ inline int swz_f(int r) { return (r & 8) | ((r & 3) << 1) | (((r >> 2) ^ (r >> 3)) & 1); }

// Byte of 16-byte chunk c of row r of a 128-token page's K or V^T: chunks 0..7 and
// 8..15 of every row are two blocks of 128-byte rows, 16 KB apart.
__device__ inline uint32_t page_chunk(int r, int c) { return uint32_t((c >> 3) * 16384 + r * 128 + (c & 7) * 16); }

// LDS byte offset of bf16 element (r, c) of a tile.
__device__ inline uint32_t swz_elem(int r, int c) {
  return uint32_t(r * 256 + ((swz_perm(c >> 3) ^ swz_f(r & 15)) << 4) + (c & 7) * 2);
}

// MFMA operand (A or B: lane l holds row/column l%32 and k-slots 8*(l/32)+e)
// from a swizzled tile stored k-major: tile row krow(kappa) holds k-slot kappa,
// and the operand's rows/columns are tile columns col0 .. col0+31.  Two
// transposing reads: in every group of 16 lanes, lane i receives element i%4
// of the 8-byte pieces read by lanes i/4 + 4k (k = 0..3), so lane r' of group g
// reads tile row krow(8*hl + 4*h + r'/4), columns col0 + 16g + 4*(r'%4) .. +3.
template <class KRow>
__device__ inline bf16x8 tr_operand(const lds_u8* tile, int col0, int lane, KRow krow) {
  const int rp = lane & 15, g = (lane >> 4) & 1, hl = lane >> 5;
  const int c = col0 + 16 * g + 4 * (rp & 3);
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (lds_v4i16*)(tile + swz_elem(krow(8 * hl + (rp >> 2)), c)));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (lds_v4i16*)(tile + swz_elem(krow(8 * hl + 4 + (rp >> 2)), c)));
  const v4i16 v[2] = {lo, hi};
  return __builtin_bit_cast(bf16x8, v);
}

// Per-lane parts of operand addresses, computed once per kernel so that every
// read in the loops is a fixed register plus a compile-time offset.
//
// TrTable: transposing reads from a k-major tile whose k-slot kappa of a
// 16-row step starting at row R (a multiple of 16) is row R + kappa
// (natural) or R + swap23(kappa) (SWAP); t[h][cb] is the byte offset, minus
// R*256, of read h of the operand over columns 32*cb .. 32*cb + 31.
struct TrTable {
  uint32_t t[2][4];
};
template <bool SWAP>
__device__ inline TrTable tr_table(int lane) {
  const int rp = lane & 15, g = (lane >> 4) & 1, hl = lane >> 5;
  TrTable T;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const int lrow = SWAP ? 8 * h + 4 * hl + (rp >> 2) : 8 * hl + 4 * h + (rp >> 2);
      T.t[h][cb] = swz_elem(lrow, 32 * cb + 16 * g + 4 * (rp & 3));
    }
  return T;
}
// LDS reads by byte address (an address of zero is an ordinary one).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
__device__ inline u32x4 lds_read16(uint32_t at) { return *(const lds_u32x4*)(uintptr_t)at; }
__device__ inline f32x4 lds_read4f(uint32_t at) { return *(const lds_f32x4*)(uintptr_t)at; }
__device__ inline v4i16 lds_read_tr(uint32_t at) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(uintptr_t)at);
}
// The operand, with the tile's LDS address added to the table.
__device__ inline bf16x8 tr_op_at(const TrTable& T, int R, int cb) {
  const v4i16 v[2] = {lds_read_tr(T.t[0][cb] + uint32_t(R * 256)), lds_read_tr(T.t[1][cb] + uint32_t(R * 256))};
  return __builtin_bit_cast(bf16x8, v);
}
// RowTable: 16-byte row reads of an A/B operand (lane holds row R + rl, rl = ln
// or swap23(ln), R a multiple of 32; dims 16ks + 8hl .. +7): u[ks] is the
// byte offset minus R*256.
struct RowTable {
  uint32_t u[8];
};
template <bool SWAP>
__device__ inline RowTable row_table(int lane) {
  const int ln = lane & 31, hl = lane >> 5;
  const int rl = SWAP ? swap23(ln) : ln;
  RowTable U;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) U.u[ks] = swz_elem(rl, 16 * ks + 8 * hl);
  return U;
}

// ---------------------------------------------------------------- dkdv ----

// One workgroup per window key tile, T/16 waves (eight for 128-token tiles):
// wave w < T/32 (group 0) and wave w + T/32 (group 1) share keys
// 32w + swap23(ln) (lane ln), so that the V operand read transposed from the
// pool's V^T tile (whose columns hold the keys in swap23 order) lands in natural
// lane order.  The kept query tiles are gathered first (mask bits) as a list of
// units of T/2 queries (half tiles; a half without a valid query gives none).
// Per unit, group 0 computes S = Q K^T and P, hands P (bf16, already in the
// B-operand layout) to its partner through LDS and accumulates dV^T += dO^T P;
// group 1 computes dP = dO V^T and, one unit later, dS = P (dP - delta) and
// dK^T += Q^T dS.  The S and dP accumulators start from the workspace's
// -LSE/scale and -delta, so P = exp2(c2 S') and dS = P dP' need no subtraction.
//
// What bounds it: four products per pair on the matrix cores, under the power
// limit (the clock falls as they get busier).  With five steps per query tile,
// the first and last half empty, and each operand read right before its
// product, they were busy 51 % of the cycles at 1.98 GHz and the 1K window (12
// heads, 24,480-token chunks, 55 % kept) took 19.2 ms; with the phases below
// 63 % at 1.76 GHz, 17.4 ms.  (The phases alone, in the compiler's order of
// reads: 47 %, 20.0 ms; with the reads ahead 59 %, 18.1 ms; the copies between
// the products instead of at the start of the phase: 63 %.)
//
// Phases.  Phase s is unit s for group 0 and for group 1's dP, unit s-1 for
// group 1's dS and dK, with one workgroup barrier after it; both groups issue
// the same number of MFMAs in it, and one SIMD runs one wave of each.  Units
// follow one another without a drain between query tiles.  Q rows live in a ring
// of four units (s-1, s, s+1 and the one being copied), dO rows in a ring of
// three, so that a unit is requested two phases before it is used.
constexpr int kQRing = 4, kORing = 3, kLRing = 4;
constexpr int kAhead = 4;   // operands in flight ahead of their product

// The rows of a unit: W = T/16 waves fill UQ = T/2 rows of 256 bytes; copy i of
// wave w fills LDS chunks [64*(W i + w), +64), rows 4(W i + w) + lane/16, whose
// low four bits do not depend on i.
__device__ inline uint32_t copy_offset8(int wave, int lane) {
  const int r = 4 * wave + (lane >> 4);
  return uint32_t(r * 256 + swz_perm((lane & 15) ^ swz_f(r & 15)) * 16);
}
// The V^T of a 64-token page ([128 dims][64 keys], 128-byte rows) into the
// swizzled [128][128] tile layout, of which it fills the first 64 columns,
// with four waves: copy i of wave w fills rows 16i + 4w + lane/16.  A lane
// whose LDS position holds one of the unused columns 64..127 fetches a
// duplicate of a used chunk of its row (in bounds, never read).
__device__ inline uint32_t copy_offset_vt64(int wave, int lane) {
  const int r = 4 * wave + (lane >> 4);
  return uint32_t(r * 128 + (swz_perm((lane & 15) ^ swz_f(r)) & 7) * 16);
}
__device__ inline void copy_vt64_w4(const uint8_t* src, uint32_t lds_tile, uint32_t voff, int wave) {
#pragma unroll
  for (int i = 0; i < 8; ++i) dma16(src + i * 2048, voff, lds_tile + uint32_t(wave) * 1024u + uint32_t(i) * 4096u);
}
__device__ inline uint32_t copy_offset8_page(int wave, int lane) {
  const int r = 4 * wave + (lane >> 4);
  return page_chunk(r, swz_perm((lane & 15) ^ swz_f(r & 15)));
}
__device__ inline void copy_tile8_page(const uint8_t* src, uint32_t lds_tile, uint32_t voff, int wave) {
#pragma unroll
  for (int i = 0; i < 4; ++i) dma16(src + i * 4096, voff, lds_tile + uint32_t(wave) * 1024u + uint32_t(i) * 8192u);
}

// dma16 of the lanes in `mask` only (the whole wave is active around it).
__device__ inline void dma16_low(const void* base, uint32_t off, uint32_t lds, uint64_t mask) {
  asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
               : : "v"(off), "s"(base), "s"(lds), "s"(mask) : "memory");
}

template <int T>
__global__ __launch_bounds__(4 * T, 2) void bwd_dkdv_kernel(BwdArgs a) {
  constexpr int kKW = T / 32;                        // key blocks = waves of a group
  constexpr int W = 2 * kKW;                         // waves
  constexpr int UQ = T / 2;                          // queries of a unit
  constexpr int NB = UQ / 32;                        // 32-query blocks of a unit
  constexpr uint32_t UB = UQ * 256;                  // bytes of a unit's Q (or dO) rows
  constexpr int kCopies = UB / 1024 / W;             // copies of a wave per unit and operand
  __shared__ uint4 sQ[kQRing][UQ * 16];
  __shared__ uint4 sO[kORing][UQ * 16];
  __shared__ uint4 sP[2][kKW][NB * 2][64];           // P operands of a unit: [parity][wave pair][block, kk][lane]
  __shared__ float sLD[kLRing][2 * kT];              // the tile's -LSE/scale, then -delta, per unit
  __shared__ uint16_t sList[2 * kBwdMaxQTiles];      // (query tile << 1) | half
  __shared__ int sN;

  // the current chunk's tiles first: they (and the pinned chunk's, next at
  // position 0) are kept by every query tile and run longest
  const int rows = a.B * a.H * a.NT;
  const int order = int(blockIdx.x) / rows;
  const int kj = xcd_deal(int(blockIdx.x) - order * rows, rows, rows, rows, rows * a.n_live, a.NT, T == 128 ? 256 : 512,
                          a.counts);
  const int t = kj % a.NT;
  const int bh = kj / a.NT;
  const int pos = order == 0 ? a.n_live - 1 : order - 1;
  const int h = bh % a.H, b = bh / a.H;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / kKW, kw = wave % kKW;
  const int lane = tid & 63, hl = lane >> 5, ln = lane & 31;
  const int kvalid = tile_valid(a.tv, t, a.NT, a.tail, T);
  const int key = kw * 32 + swap23(ln);         // this lane's key (result column)
  const bool key_ok = key < kvalid;
  const int j = pos * a.NT + t;                 // logical key tile
  const uint8_t* qbase = a.work + size_t(bh) * a.NT * kBwdQTile;

  // B operands of the wave's keys: group 0 K rows from the page, group 1 V
  // read transposed from the page's V^T, staged in the P slots (128-token
  // tiles) or in the Q ring (64-token tiles, before any unit is copied)
  const uint8_t* page = a.pool + ((size_t(a.slot_of[pos]) * a.B * a.H + bh) * a.NT + t) * page_bytes(T, kD);
  bf16x8 bop[8];
  if (grp == 0) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint32_t off = T == 128 ? page_chunk(key, 2 * ks + hl) : uint32_t(key * 256 + (2 * ks + hl) * 16);
      bop[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(page + off));
    }
  }
  static_assert(T == 128 ? sizeof(sP) == kTile : sizeof(sQ) == kTile, "V^T stage");
  uint4* const stage = T == 128 ? &sP[0][0][0][0] : &sQ[0][0];
  if constexpr (T == 128)
    copy_tile8_page(page + kTile, lds_addr(stage), copy_offset8_page(wave, lane), wave);
  else
    copy_vt64_w4(page + T * kD * 2, lds_addr(stage), copy_offset_vt64(wave, lane), wave);

  // units of the kept query tiles, ascending
  if (wave == 0) {
    int cnt = 0;
    for (int base = 0; base < a.NT; base += 512) {
      uint32_t w[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = base + 64 * k + lane;
        w[k] = i < a.NT ? a.mask[size_t(bh * a.NT + i) * a.mask_words + (j >> 5)] : 0u;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = base + 64 * k + lane;
        int n = 0;
        if ((w[k] >> (j & 31)) & 1u) {
          const int v = tile_valid(a.tv, i, a.NT, a.tail, T);
          n = v > UQ ? 2 : (v > 0 ? 1 : 0);
        }
        const uint64_t b1 = __ballot(n >= 1), b2 = __ballot(n == 2);
        const uint64_t below = (uint64_t(1) << lane) - 1;
        const int at = cnt + __popcll(b1 & below) + __popcll(b2 & below);
        if (n >= 1) sList[at] = uint16_t(i << 1);
        if (n == 2) sList[at + 1] = uint16_t((i << 1) | 1);
        cnt += __popcll(b1) + __popcll(b2);
      }
    }
    if (lane == 0) sN = cnt;
  }
  meet<0>();
  const int U = __builtin_amdgcn_readfirstlane(sN);

  // Copies of unit n (list entry e): Q and dO rows, and by wave 0 the tile's
  // per-query values.
  const uint32_t voff = copy_offset8(wave, lane);
  const uint32_t lq0 = lds_addr(&sQ[0][0]), lo0 = lds_addr(&sO[0][0]), ll0 = lds_addr(&sLD[0][0]);
  // Past the end the last unit is copied again, into a slot that nothing reads
  // any more: every phase issues the same copies, without a branch.
  struct Source {
    const uint8_t* rec;
    uint32_t half, qslot, oslot;
  };
  auto entry = [&](int n) { return uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(sList[min(n, U - 1)]))); };
  auto source = [&](uint32_t e, uint32_t qslot, uint32_t oslot) {
    return Source{qbase + size_t(e >> 1) * kBwdQTile, (e & 1) * UB, qslot, oslot};
  };
  constexpr int kIssue = 2 * kCopies + 1;       // copies of a wave per unit
  auto issue = [&](const Source& c, int k) {    // copy k of them
    if (k == 2 * kCopies) {
      constexpr uint32_t part = 2 * kT * 4 / W; // this wave's share of the per-query values
      dma16_low(c.rec + 2 * kTile + uint32_t(wave) * part, uint32_t(lane) * 16u,
                ll0 + c.qslot * uint32_t(sizeof(sLD[0])) + uint32_t(wave) * part, (uint64_t(1) << (part / 16)) - 1);
      return;
    }
    const uint32_t at = uint32_t(k >> 1) * W * 1024u;
    dma16(c.rec + (k & 1) * kTile + c.half + at, voff,
          ((k & 1) ? lo0 + c.oslot * UB : lq0 + c.qslot * UB) + uint32_t(wave) * 1024u + at);
  };
  auto issue_all = [&](const Source& c) {
#pragma unroll
    for (int k = 0; k < kIssue; ++k) issue(c, k);
  };
  uint32_t e0 = 0, e1 = 0, e2 = 0;
  if (U > 0) {
    e0 = entry(0);
    e1 = entry(1);
    e2 = entry(2);
  }
  if (T == 128 && U > 0) {                      // the stage is outside the rings
    issue_all(source(e0, 0, 0));
    issue_all(source(e1, 1, 1));
  }
  if (grp == 1) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      bop[ks] = tr_operand((const lds_u8*)stage, kw * 32, lane, [&](int kap) { return 16 * ks + kap; });
  }
  if (T == 64 && U > 0) {
    meet<0>();                                  // V^T consumed
    issue_all(source(e0, 0, 0));
    issue_all(source(e1, 1, 1));
  }

  f32x16 acc[4];                                // dV^T (group 0) or dK^T (group 1): [dim block][32 dims x 32 keys]
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) acc[mb] = f32x16{};
  const float c2 = a.scale_log2;
  const float pad = key_ok ? 0.f : -INFINITY;   // padding keys (lanes) weigh nothing; no branch in the phase
  uint4* const pslot = &sP[0][kw][0][lane];     // this wave pair's P operands
  constexpr uint32_t kPStep = sizeof(sP[0]) / 16;
  // Operand addresses within the current ring slots, advanced once per phase:
  // tr: transposing reads (X^T: k-slot kappa = query 16kk + swap23(kappa)) of
  // dO (group 0) or Q (group 1); rt: row reads (X rows: query ln of a block) of
  // Q (group 0) or dO (group 1); ld: the per-query seeds of the row reads.
  TrTable tr = tr_table<true>(lane);
  RowTable rt = row_table<false>(lane);
  {
    const uint32_t bt = grp == 0 ? lo0 : lq0, br = grp == 0 ? lq0 : lo0;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) tr.t[k][cb] += bt;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) rt.u[ks] += br;
  }
  const uint32_t ld0 = ll0 + uint32_t(16 * hl + (grp == 0 ? 0 : 4 * kT));

  // A unit's products of one wave: 8 NB row products (X K^T or X V^T, chain
  // qb over ks), then 8 NB transposed ones (acc^T += X^T op, block qb, step kk,
  // dims 32 mb ..).  Product i and its operand, read kAhead products earlier.
  constexpr int kRows = 8 * NB, kAll = 16 * NB;
  auto load = [&](int i) -> bf16x8 {
    if (i < kRows) return __builtin_bit_cast(bf16x8, lds_read16(rt.u[i & 7] + uint32_t((i >> 3) * 32 * 256)));
    const int k = i - kRows;
    return tr_op_at(tr, 16 * (k >> 2), k & 3);
  };
  auto row_product = [&](int i, const bf16x8& x, f32x16 (&v)[NB]) {
    v[i >> 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, bop[i & 7], v[i >> 3], 0, 0, 0);
  };
  auto tr_product = [&](int i, const bf16x8& x, const bf16x8 (&op)[NB][2]) {
    const int k = i - kRows, mb = k & 3;
    acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, op[k >> 3][(k >> 2) & 1], acc[mb], 0, 0, 0);
  };
  // The row products start from the per-query terms, in the result layout:
  // register 4g + e = query qb*32 + 8g + 4hl + e.
  auto seed = [&](uint32_t ld, f32x16 (&v)[NB]) {
#pragma unroll
    for (int qb = 0; qb < NB; ++qb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 c4 = lds_read4f(ld + uint32_t(4 * (qb * 32 + 8 * g)));
        v[qb][4 * g] = c4.x;
        v[qb][4 * g + 1] = c4.y;
        v[qb][4 * g + 2] = c4.z;
        v[qb][4 * g + 3] = c4.w;
      }
  };
  // Two elements (registers 2e, 2e+1) of a block's operand.
  auto put = [&](bf16x8 (&op)[2], int e, float x0, float x1) {
    op[e >> 2][2 * (e & 3)] = (__bf16)x0;
    op[e >> 2][2 * (e & 3) + 1] = (__bf16)x1;
  };
  auto advance = [&](uint32_t (&x)[8], bool wrap, int ring) {
    const uint32_t d = wrap ? uint32_t(-(ring - 1) * int(UB)) : UB;
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] += d;
  };
  auto advance_tr = [&](bool wrap, int ring) {
    const uint32_t d = wrap ? uint32_t(-(ring - 1) * int(UB)) : UB;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) tr.t[k][cb] += d;
  };

  // Scheduling fences pin the order written here: a product, the read of a
  // later one's operand, a piece of vector work.  Left to itself the compiler
  // reads each operand right before its product and runs the vector work
  // between them, so that a product waits for an LDS round trip.
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  constexpr int kGap = kAll / kIssue;           // products between two of the next unit's copies
  // Group 0, unit s: S, P, the P slot, dV.  The weights of a block are formed
  // beside the next block's products.
  auto unit0 = [&](uint32_t ld, uint32_t par, const Source& next) {
    f32x16 sv[NB];
    bf16x8 op[NB][2], x[kAll];
    seed(ld, sv);                               // -LSE/scale (-inf on padding queries)
#pragma unroll
    for (int i = 0; i < kAhead; ++i) x[i] = load(i);
    auto weights = [&](int qb, int e) {
      put(op[qb], e, __builtin_amdgcn_exp2f(__builtin_fmaf(sv[qb][2 * e], c2, pad)),
          __builtin_amdgcn_exp2f(__builtin_fmaf(sv[qb][2 * e + 1], c2, pad)));
      if ((e & 3) == 3) pslot[par * kPStep + (qb * 2 + (e >> 2)) * 64] = __builtin_bit_cast(uint4, op[qb][e >> 2]);
    };
    fence();
#pragma unroll
    for (int i = 0; i < kAll; ++i) {
      if (i < kRows) row_product(i, x[i], sv);
      else tr_product(i, x[i], op);
      if (i + kAhead < kAll) x[i + kAhead] = load(i + kAhead);
      if (i >= 8 && i < kAll - 8) weights((i - 8) >> 3, i & 7);
      if (NB == 1 && i == 7) {                  // one block: nothing to run beside
#pragma unroll
        for (int e = 0; e < 8; ++e) weights(0, e);
      }
      if (i % kGap == kGap - 1 && i / kGap < kIssue) issue(next, i / kGap);
      fence();
    }
  };
  // Group 1: dP - delta of a unit (kDp) into nv, and dS (from the P slot and
  // the dP of the unit before, ov) and dK of that unit (kDk).
  auto unit1 = [&](auto dp, auto dk, uint32_t ld, uint32_t par, const f32x16 (&ov)[NB], f32x16 (&nv)[NB],
                   const Source& next) {
    constexpr bool kDp = decltype(dp)::value, kDk = decltype(dk)::value;
    constexpr int i0 = kDp ? 0 : kRows, i1 = kDk ? kAll : kRows;
    bf16x8 pk[NB][2], op[NB][2], x[kAll];
    if (kDk) {
#pragma unroll
      for (int qb = 0; qb < NB; ++qb)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
          pk[qb][kk] = __builtin_bit_cast(bf16x8, pslot[par * kPStep + (qb * 2 + kk) * 64]);
    }
    if (kDp) seed(ld, nv);                      // -delta
#pragma unroll
    for (int i = i0; i < i0 + kAhead; ++i) x[i] = load(i);
    auto ds = [&](int qb, int e) {              // k-slot of operand kk: result register 8kk + slot
      put(op[qb], e, float(pk[qb][e >> 2][2 * (e & 3)]) * ov[qb][2 * e],
          float(pk[qb][e >> 2][2 * (e & 3) + 1]) * ov[qb][2 * e + 1]);
    };
    fence();
    if (kDk && !kDp) {
#pragma unroll
      for (int k = 0; k < kRows; ++k) ds(k >> 3, k & 7);
    }
#pragma unroll
    for (int i = i0; i < i1; ++i) {
      if (i < kRows) row_product(i, x[i], nv);
      else tr_product(i, x[i], op);
      if (i + kAhead < i1) x[i + kAhead] = load(i + kAhead);
      if (kDk && i < kRows) ds(i >> 3, i & 7);
      if (kDp && kDk && i % kGap == kGap - 1 && i / kGap < kIssue) issue(next, i / kGap);
      fence();
    }
  };

  // Each group runs its own copy of the phase loop (same meetings in the same
  // order), so that no branch on the group sits inside it.
  auto run = [&](auto group) {
    constexpr int G = decltype(group)::value;
    f32x16 dpv[NB];
    uint32_t om = 0;                            // s % 3
    auto phase = [&](int s, auto first) {
      constexpr bool kFirst = decltype(first)::value;
      // unit s has landed; the slots of unit s+2 are free
      const Source next = source(e2, uint32_t(s + 2) & 3u, om == 0 ? 2u : om - 1u);
      const uint32_t ld = ld0 + (uint32_t(s) & 3u) * uint32_t(sizeof(sLD[0])) + (e0 & 1u) * uint32_t(4 * UQ);
      const uint32_t e3 = sList[min(s + 3, U - 1)];
      if constexpr (G == 0) {
        unit0(ld, uint32_t(s) & 1u, next);
        advance(rt.u, (s & 3) == 3, kQRing);
        advance_tr(om == 2, kORing);
      } else {
        f32x16 nv[NB];
        if constexpr (kFirst) issue_all(next);
        unit1(std::true_type{}, std::bool_constant<!kFirst>{}, ld, uint32_t(s - 1) & 1u, dpv, nv, next);
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) dpv[qb] = nv[qb];
        if constexpr (!kFirst) advance_tr((s & 3) == 0, kQRing);
        advance(rt.u, om == 2, kORing);
      }
      om = om == 2 ? 0 : om + 1;
      meet<kIssue>();                           // unit s+1 has landed; unit s+2 may be in flight
      e0 = e1;
      e1 = e2;
      e2 = __builtin_amdgcn_readfirstlane(e3);
    };
    meet<kIssue>();                             // unit 0 has landed, unit 1 may be in flight
    phase(0, std::true_type{});
    for (int s = 1; s < U; ++s) phase(s, std::false_type{});
    if constexpr (G == 1) {
      f32x16 nv[NB];
      unit1(std::false_type{}, std::true_type{}, 0, uint32_t(U - 1) & 1u, dpv, nv, Source{});
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // no copy outlives the workgroup
  };

  if (U > 0) {
    if (grp == 0) run(std::integral_constant<int, 0>{});
    else run(std::integral_constant<int, 1>{});
  }

  // store: lane holds key `key`, dims mb*32 + 8*(r/4) + 4*hl + r%4; padding
  // rows inside the chunk (block order) get zeros
  const size_t tok = size_t(t) * T + key;
  if (tok < size_t(a.L)) {
    float* dst = (grp ? a.dk : a.dv) + (((size_t(pos) * a.B + b) * a.L + tok) * a.H + h) * kD;
    const float f = grp ? a.scale : 1.0f;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(dst + mb * 32 + 8 * g + 4 * hl) =
            key_ok ? make_float4(acc[mb][4 * g] * f, acc[mb][4 * g + 1] * f, acc[mb][4 * g + 2] * f,
                                 acc[mb][4 * g + 3] * f)
                   : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// ------------------------------------------------------------------ dq ----

// One workgroup of four waves per query tile, two workgroups per CU.  The row's
// list is walked in units of 64 keys (half of a 128-token tile; a half without
// a valid key gives none).  128-token tiles: wave w holds queries 32w .. and
// takes both 32-key blocks of a unit.  64-token tiles: wave w holds queries
// 32 (w % 2) .. and takes key block w / 2; the two key blocks' dQ are added
// through LDS at the end.
//
// Per key block: S^T = K Q^T, dP^T = V dO^T, dS^T, dQ^T += K^T dS^T.  The S^T and
// dP^T result rows of a block hold keys swap23(m) of it (m = result row), the
// order in which the V operand arrives when read transposed from the page's
// V^T; K rows are read in the same order.  dS^T as a B operand then holds natural
// key order.
//
// A unit is 32 KB of LDS, in 128-byte rows: K as two blocks of 64 dimensions
// ([2][64 keys][64]), V^T as [128 dimensions][64 keys].  16-byte chunk c of K row
// r sits at position c ^ f(r), f = (r1, r2 ^ r0, r3); of V^T row r at
// c ^ 2 (r % 4).  Row reads (f runs through all eight values over the rows of
// equal parity of any sixteen, and over rows 0..3 and 8..11) and transposing
// reads (four consecutive rows, 64 bytes each) are free of bank conflicts, with
// 32 or 64 banks, and a lane needs four addresses for K rows, four for K^T and
// one per key block for V: the rest are compile-time offsets.
//
// What bounds it: three products per pair on the matrix cores, under the power
// limit.  A whole page per step, copied into the only buffer between two
// barriers, left a workgroup without work for the length of a copy; now the
// next unit is copied, between the products, while one is used, one barrier per
// unit, with the order of products, reads ahead and vector work written out as
// in dkdv.  1K window: 13.8 -> 12.3 ms, the matrix cores busy 76 % of the cycles
// at 1.55 GHz (58 % at 1.81 before).  64-token tiles had two waves a workgroup
// and one per SIMD; with four and the keys shared 160 -> 80 us (batch 2, 6 heads,
// 1,531 tokens, three chunks).
constexpr int kDqList = 1024;                  // list entries taken into LDS at a time

__device__ inline int swz_k(int r) { return ((r & 2) << 1) | (((r >> 1) ^ (r << 1)) & 2) | ((r >> 3) & 1); }

template <int T>
__global__ __launch_bounds__(256, 2) void bwd_dq_kernel(BwdArgs a) {
  constexpr int NB = T / 64;                   // key blocks of a wave per unit
  constexpr uint32_t kUnit = 32768;
  __shared__ uint4 sbuf[2][kUnit / 16];        // K 16 KB, V^T 16 KB
  __shared__ uint32_t sunit[2 * kDqList + 1];  // (key tile << 1) | half; the count last

  const int rows = a.B * a.H * a.NT;
  const int row = xcd_deal(int(blockIdx.x), rows, rows, rows, rows, a.NT, 512, a.counts);   // (b*H + h)*NT + i
  const int i = row % a.NT;
  const int bh = row / a.NT;
  const int h = bh % a.H, b = bh / a.H;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hl = lane >> 5, ln = lane & 31, rp = lane & 15, g = (lane >> 4) & 1;
  const int qw = T == 128 ? wave : wave & 1;   // query block
  const int kw = T == 128 ? 0 : wave >> 1;     // first key block
  const int q = qw * 32 + ln;                  // this lane's query (result column)

  const uint8_t* rec = a.work + size_t(row) * kBwdQTile;
  bf16x8 qf[8], of[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    qf[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(rec + size_t(q) * 256 + (2 * ks + hl) * 16));
    of[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(rec + kTile + size_t(q) * 256 + (2 * ks + hl) * 16));
  }
  const float c2 = a.scale_log2;
  // the lane's query terms: P = exp2(c2 S - LSE log2(e)) (-inf on padding
  // queries), and -delta as the seed of the dP products
  const float nl = reinterpret_cast<const float*>(rec + 2 * kTile)[q] * c2;
  const float nd = reinterpret_cast<const float*>(rec + 2 * kTile)[kT + q];
  f32x16 negd;
#pragma unroll
  for (int r = 0; r < 16; ++r) negd[r] = nd;

  // operand addresses in the current buffer
  const uint32_t lds0 = lds_addr(&sbuf[0][0]);
  uint32_t kr[4], kt[2][2], vt[NB];
  {
    const int rr = swap23(ln);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      kr[k] = lds0 + uint32_t(kw * 4096 + rr * 128 + 16 * ((2 * k + hl) ^ swz_k(rr & 15)));
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int r = 8 * hl + 4 * hh + (rp >> 2);
        kt[hh][m] = lds0 + uint32_t(kw * 4096 + r * 128 + 16 * ((4 * m + 2 * g + ((rp >> 1) & 1)) ^ swz_k(r)) + 8 * (rp & 1));
      }
#pragma unroll
    for (int n = 0; n < NB; ++n)
      vt[n] = lds0 + uint32_t(16384 + (8 * hl + (rp >> 2)) * 128 +
                              16 * ((4 * (kw + n) + 2 * g + ((rp >> 1) & 1)) ^ (2 * (rp >> 2))) + 8 * (rp & 1));
  }
  // Copies: copy t of wave w for K fills block t/2, rows 8 (w + 4 (t%2)) + lane/8;
  // for V^T rows 8 (w + 4t) + lane/8.
  constexpr uint32_t kRowStep = T == 128 ? 128 : 256, kBlock = T == 128 ? 16384 : 128;
  const uint32_t koff = uint32_t((lane >> 3) * kRowStep + 16 * ((lane & 7) ^ swz_k(8 * (wave & 1) + (lane >> 3))));
  const uint32_t voff = uint32_t((lane >> 3) * 128 + 16 * ((lane & 7) ^ (2 * ((lane >> 3) & 3))));
  const size_t pbytes = page_bytes(T, kD);
  const uint8_t* head_pages = uniform_ptr(a.pool + size_t(bh) * a.NT * pbytes);
  const size_t slot_stride = size_t(a.B) * a.H * a.NT * pbytes;
  const int N = ((const const_i32*)a.counts)[row];
  const int32_t* list = a.idx + size_t(row) * a.nk_cap;

  f32x16 dqt[4];                                // [4 dim blocks][32 dims x 32 queries]
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) dqt[mb] = f32x16{};

  struct Unit {
    const uint8_t* k;      // its K rows
    const uint8_t* v;      // and V^T rows
    int valid;             // valid keys
  };
  auto unit = [&](uint32_t x) {
    const int half = int(x & 1u);
    const int pos = div_nt(x >> 1, a.nt_div);
    const int t = int(x >> 1) - pos * a.NT;
    const uint8_t* page = head_pages + size_t(a.slot_of[pos]) * slot_stride + size_t(t) * pbytes;
    return Unit{page + half * 64 * kRowStep, page + T * kD * 2 + 16384 * half,
                min(tile_valid(a.tv, t, a.NT, a.tail, T) - 64 * half, 64)};
  };
  auto issue = [&](const Unit& u, uint32_t buf, int k) {
    const int t = k & 3;
    const uint32_t dst = lds0 + buf * kUnit + uint32_t(wave) * 1024u;
    if (k < 4)
      dma16(u.k + (t >> 1) * kBlock + uint32_t(8 * (wave + 4 * (t & 1))) * kRowStep, koff, dst + uint32_t(t) * 4096u);
    else
      dma16(u.v + uint32_t(wave + 4 * t) * 1024u, voff, dst + 16384u + uint32_t(t) * 4096u);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

  // Products of a unit: per key block n S (0..7), dP (8..15); then per block dQ.
  // With two blocks: S0, dP0, S1, dP1, dQ0, dQ1.
  constexpr int kAll = 24 * NB, kSP = 16 * NB;
  constexpr int kReads = 5;                     // operands in flight: what the registers hold
  auto load = [&](int k) -> bf16x8 {
    if (k < kSP) {
      const int n = k >> 4, ks = k & 7;
      if ((k & 8) == 0)
        return __builtin_bit_cast(bf16x8, lds_read16(kr[ks & 3] + uint32_t(n * 4096 + (ks >> 2) * 8192)));
      const v4i16 v[2] = {lds_read_tr(vt[n] + uint32_t(ks * 2048)), lds_read_tr(vt[n] + uint32_t(ks * 2048 + 512))};
      return __builtin_bit_cast(bf16x8, v);
    }
    const int m = k - kSP, n = m >> 3, kk = (m >> 2) & 1, mb = m & 3;
    const uint32_t at = uint32_t(n * 4096 + kk * 2048 + (mb >> 1) * 8192);
    const v4i16 v[2] = {lds_read_tr(kt[0][mb & 1] + at), lds_read_tr(kt[1][mb & 1] + at)};
    return __builtin_bit_cast(bf16x8, v);
  };
  auto body = [&](const Unit& cur, const Unit& next, uint32_t nbuf) {
    f32x16 sv[NB], dp[NB];
    bf16x8 op[NB][2], x[kAll];
    // keys past the unit's valid ones weigh nothing (a rare case: their indices
    // are formed here, not held across the loop)
    auto mask = [&](int n) {
      if (cur.valid < 64) {
        int h4 = 4 * hl;
        asm volatile("" : "+v"(h4));
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if ((kw + n) * 32 + swap23(8 * (r >> 2) + h4 + (r & 3)) >= cur.valid) sv[n][r] = -INFINITY;
      }
    };
    auto weight = [&](int n, int r) { sv[n][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[n][r], c2, nl)); };
    auto ds = [&](int n, int e) {
      op[n][e >> 2][2 * (e & 3)] = (__bf16)(sv[n][2 * e] * dp[n][2 * e]);
      op[n][e >> 2][2 * (e & 3) + 1] = (__bf16)(sv[n][2 * e + 1] * dp[n][2 * e + 1]);
    };
#pragma unroll
    for (int k = 0; k < kReads; ++k) x[k] = load(k);
    fence();
    auto eight = [&](auto first) {              // products first .. first + 7
      constexpr int k0 = decltype(first)::value;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = k0 + j;
        if constexpr (k0 < kSP) {
          const int n = k0 >> 4;
          if constexpr ((k0 & 8) == 0)
            sv[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[k], qf[j], j ? sv[n] : f32x16{}, 0, 0, 0);
          else
            dp[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[k], of[j], j ? dp[n] : negd, 0, 0, 0);
        } else {
          dqt[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[k], op[(k0 - kSP) >> 3][j >> 2], dqt[j & 3], 0, 0, 0);
        }
        if (k + kReads < kAll) x[k + kReads] = load(k + kReads);
        if constexpr (k0 < kSP && (k0 & 8) != 0) {   // beside dP of a block: its weights
          weight(k0 >> 4, 2 * j);
          weight(k0 >> 4, 2 * j + 1);
        }
        if constexpr (NB == 2 && k0 == 16) ds(0, j);   // beside S of block 1
        if constexpr (NB == 2 && k0 == 32) ds(1, j);   // beside dQ of block 0
        if (k % 2 == 1 && k < 16) issue(next, nbuf, k >> 1);   // the next unit's copies
        fence();
      }
      // what was formed here stays here (the masks' branches would let the
      // compiler sink it to where it is used)
      if constexpr (k0 < kSP && (k0 & 8) != 0) asm volatile("" : "+v"(sv[k0 >> 4]));
      if constexpr (NB == 2 && k0 == 16) asm volatile("" : "+v"(op[0][0]), "+v"(op[0][1]));
    };
    eight(std::integral_constant<int, 0>{});
    mask(0);
    eight(std::integral_constant<int, 8>{});
    if constexpr (NB == 2) {
      eight(std::integral_constant<int, 16>{});
      mask(1);
      eight(std::integral_constant<int, 24>{});
      eight(std::integral_constant<int, 32>{});
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) ds(0, e);
    }
    eight(std::integral_constant<int, kAll - 8>{});
  };

  for (int base = 0; base < N; base += kDqList) {
    // the units of the next kDqList entries; entries naming a tile outside the
    // window (stale lists) count no key
    if (base > 0) meet<0>();                    // the table is no longer read
    if (wave == 0) {
      int cnt = 0;
      const int end = min(N, base + kDqList);
      for (int e0 = base; e0 < end; e0 += 256) {
        uint32_t jj[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int e = e0 + 64 * k + lane;
          jj[k] = e < end ? uint32_t(list[e]) : 0xffffffffu;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t j = jj[k];
          int n = 0;
          if (j < uint32_t(a.nk)) {
            const int v = tile_valid(a.tv, int(j % uint32_t(a.NT)), a.NT, a.tail, T);
            n = v > 64 ? 2 : (v > 0 ? 1 : 0);
          }
          const uint64_t b1 = __ballot(n >= 1), b2 = __ballot(n == 2);
          const uint64_t below = (uint64_t(1) << lane) - 1;
          const int at = cnt + __popcll(b1 & below) + __popcll(b2 & below);
          if (n >= 1) sunit[at] = j << 1;
          if (n == 2) sunit[at + 1] = (j << 1) | 1u;
          cnt += __popcll(b1) + __popcll(b2);
        }
      }
      if (lane == 0) sunit[2 * kDqList] = uint32_t(cnt);
    }
    meet<0>();
    const int U = __builtin_amdgcn_readfirstlane(sunit[2 * kDqList]);
    if (U == 0) continue;
    auto entry = [&](int u) { return uint32_t(__builtin_amdgcn_readfirstlane(sunit[min(u, U - 1)])); };
    Unit cur = unit(entry(0)), next = unit(entry(1));
#pragma unroll
    for (int k = 0; k < 8; ++k) issue(cur, 0, k);
    for (int u = 0; u < U; ++u) {
      meet<0>();                                // unit u has landed; the other buffer is free
      const uint32_t x2 = sunit[min(u + 2, U - 1)];
      body(cur, next, uint32_t(u + 1) & 1u);    // past the end the last unit is copied again, and not read
      const uint32_t d = (u & 1) ? uint32_t(-int(kUnit)) : kUnit;
#pragma unroll
      for (int k = 0; k < 4; ++k) kr[k] += d;
#pragma unroll
      for (int k = 0; k < 4; ++k) kt[k >> 1][k & 1] += d;
#pragma unroll
      for (int k = 0; k < NB; ++k) vt[k] += d;
      cur = next;
      next = unit(__builtin_amdgcn_readfirstlane(x2));
    }
    if (U & 1) {                                // the next entries start in buffer 0 again
#pragma unroll
      for (int k = 0; k < 4; ++k) kr[k] -= kUnit;
#pragma unroll
      for (int k = 0; k < 4; ++k) kt[k >> 1][k & 1] -= kUnit;
#pragma unroll
      for (int k = 0; k < NB; ++k) vt[k] -= kUnit;
    }
  }
  meet<0>();                                    // no copy outlives the workgroup

  if constexpr (T == 64) {
    float* xo = reinterpret_cast<float*>(&sbuf[0][0]);   // [2 query blocks][4][16][64 lanes]
    if (kw == 1) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int e = 0; e < 16; ++e) xo[((qw * 4 + mb) * 16 + e) * 64 + lane] = dqt[mb][e];
    }
    meet<0>();
    if (kw == 1) return;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) dqt[mb][e] += xo[((qw * 4 + mb) * 16 + e) * 64 + lane];
  }
  // padding rows inside the chunk accumulated zeros (their weights are zero)
  if (size_t(i) * T + q < size_t(a.L)) {
    const size_t base = ((size_t(b) * a.L + size_t(i) * T + q) * a.H + h) * kD;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int d0 = mb * 32 + 8 * k + 4 * hl;
        *reinterpret_cast<float4*>(a.dq + base + d0) =
            make_float4(dqt[mb][4 * k] * a.scale, dqt[mb][4 * k + 1] * a.scale, dqt[mb][4 * k + 2] * a.scale,
                        dqt[mb][4 * k + 3] * a.scale);
      }
  }
}

}  // namespace

// Scratch of the no-allocation backward: the query-tile records that
// launch_attn_bwd keeps in the caller's workspace, in a file-scope device
// array instead.  Every GPU the library runs on holds its own copy until the
// process ends; in host code the array's name is only a stand-in, so kernels
// are handed its device address, looked up once per device.
static __device__ __align__(256) uint8_t scratch[kBwdScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the device of `stream` (the current device
// for the null stream), looked up with that device current on the first call.
hipError_t scratch_address(hipStream_t stream, void** out) {
  int cur = 0;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  int dev = cur;
  if (stream != nullptr && (e = hipStreamGetDevice(stream, &dev)) != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    if (dev != cur && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (dev != cur) {
      const hipError_t r = hipSetDevice(cur);
      if (e == hipSuccess) e = r;
    }
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace

hipError_t launch_attn_bwd_noalloc(BwdArgs a, hipStream_t stream) {
  if (size_t(a.B) * size_t(a.H) * size_t(a.NT) * kBwdQTile > kBwdScratchBytes) return hipErrorInvalidValue;
  void* p = nullptr;
  hipError_t e = scratch_address(stream, &p);
  if (e != hipSuccess) return e;
  a.work = static_cast<uint8_t*>(p);
  return launch_attn_bwd(a, stream);
}

namespace {

template <int T>
hipError_t launch_bwd_t(const BwdArgs& a, hipStream_t stream) {
  const unsigned qrows = unsigned(a.B) * unsigned(a.H) * unsigned(a.NT);
  const unsigned ktiles = unsigned(a.n_live) * qrows;
  bwd_prep_kernel<T><<<qrows, kThreads, 0, stream>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  bwd_dkdv_kernel<T><<<ktiles, 4 * T, 0, stream>>>(a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  bwd_dq_kernel<T><<<qrows, 256, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bwd(const BwdArgs& a, hipStream_t stream) {
  if (a.T == 128) return launch_bwd_t<128>(a, stream);
  if (a.T == 64) return launch_bwd_t<64>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace uf
