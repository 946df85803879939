// attn_fwd (64-token tiles): block-sparse chunk-causal attention forward on
// gfx950.
//
// For one (b, h, query tile i) the workgroup walks the kept key tiles of its
// list (Eq. 4: attention restricted to the kept blocks of the chunk-causal
// window) and keeps an online softmax.
//
// Work split: four waves, three workgroups per CU.  Wave (kw, qw) holds queries
// 32 qw .. of the tile and takes key block kw (32 keys) of every kept tile; the
// two key blocks keep their own (m, l, O), and at the end block 1 hands its
// state to block 0 through LDS (log-sum-exp merge).  S^T = K Q^T and
// O^T += V^T P^T on v_mfma_f32_32x32x16_bf16, K and V^T from LDS as the A operand,
// Q^T and P^T in registers as the B operand: every lane owns one query column, so
// the row max and sum need one permlane32 exchange, and the weights rounded to
// bf16 in place are the PV operand (V pages keep the keys of each group of 16 in
// swap23 order, the k-slot order of the S^T result lanes).
//
// What bounds it: a 64-token tile brings 32 KB of K and V for half the products
// of a 128-token one, so the copies (64 bytes a cycle and CU if the matrix cores
// never waited) and their latency.  Per tile a workgroup runs S, softmax and PV
// one after the other and waits for copies twice; three workgroups beside each
// other, 48 KB of LDS each (two K buffers, one V buffer), fill each other's
// waits: 12 heads, 4,665 tokens, four chunks, half of two of them kept, take
// 477 us (840 TFLOP/s); one workgroup per CU whose two groups of two waves walked
// alternate tiles in single buffers, one wave per SIMD, took 855 us (469).  The
// smallest window (6 rows of 6 tiles) takes 10.4 us, 12.1 before.
//
// Memory: pages are copied HBM -> LDS by direct global_load_lds (16 bytes per
// lane).  K lies in LDS as two blocks of 64 dimensions, V^T as one of 64 keys,
// all in 128-byte rows whose 16-byte chunks are XOR-swizzled as in the 128-token
// kernel, so that an operand read needs one of four lane addresses plus a
// compile-time offset and is free of bank conflicts.  K of the next tile and V
// of this one are requested when S begins (every wave has then finished with
// both buffers); V is waited for before PV, K before the next S.
//
// Softmax in base 2 with a lazy offset m per lane: weights exp2(c2 s - m), c2 =
// scale*log2(e).  The offset is raised, and O and l rescaled, on a wave's first
// kExact tiles and its first valid key, later only when a lane's 16 weights sum to
// more than kSumBound.  (The weight of the key that sets the offset is 1, which bf16
// holds exactly; that key is often the row's largest in a short row, and the largest
// weight's rounding is what O and LSE keep.  A wave sees 32 keys of a tile, so an
// offset from its first tile alone made rows of two tiles less exact than one from
// a tile's 64 keys: LSE by 58 %, O by 30 %, and rows of six by 10 and 7 % at logits
// of standard deviation 1.9.  With three tiles both are below it: 0.3 to 0.8 us a
// launch of one round (6 tiles 9.1 -> 9.6 us, 40 tiles 31.3 -> 32.1), none on longer
// ones, as the bound is a variable of the loop; as a flag beside it 2 %.)  The row sum
// adds the bf16-rounded weights that the PV product uses (v_dot2_f32_bf16; fp32
// adds of the unrounded ones were 0.6 % faster and raised O's error by 1 to 3 %).
// O is normalised once at the end and rounded to bf16 (nearest even).
#include "attn_common.h"

namespace uf {
namespace {

using namespace attn;

constexpr int kT = 64;
constexpr uint32_t kBuf = 16384;       // a tile's K, or its V^T
constexpr float kSumBound = 4096.0f;   // lane row-sum bound of 16 weights
constexpr int kList = 1024;            // list entries taken into LDS at a time
constexpr int kAhead = 6;              // operands in flight ahead of their product
constexpr int kExact = 3;              // first tiles of a list whose maxima always raise the offset

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
__device__ inline bf16x8 lds_operand(uint32_t at) {
  return __builtin_bit_cast(bf16x8, *(const lds_u32x4*)(uintptr_t)at);
}

// SPLIT: as in the 128-token kernel, the first a.split_from workgroups run
// rows 0 .. split_from-1 whole and every later row is cut into a.split slices
// of its list; a slice writes its unnormalised O, its offset (base-2 units)
// and its row sum to a.work for the merge.
template <bool SPLIT>
__global__ __launch_bounds__(256, 3) void attn_fwd_kernel(AttnArgs a) {
  __shared__ uint4 sbuf[3][kBuf / 16];             // K, K, V^T
  __shared__ uint32_t sunit[kList + 1];            // key tiles with a valid key; the count last

  // (the grid from the arguments that are read anyway: gridDim is another dependent
  // load at the head of the kernel, 0.5 us of a 42 us launch)
  const int rows = a.B * a.H * a.NT;
  const int grid = SPLIT ? a.split_from + (rows - a.split_from) * a.split : rows;
  int row = xcd_deal(int(blockIdx.x), grid, SPLIT ? a.split_from : rows, rows, grid, a.NT, 3 * 256, a.counts);
  int part = 0;
  bool partial = false;
  if (SPLIT && row >= a.split_from) {
    const int k = row - a.split_from;
    row = a.split_from + k / a.split;
    part = k - (row - a.split_from) * a.split;
    partial = true;
  }
  const int qt = row % a.NT;
  const int bh = row / a.NT;
  const int h = bh % a.H;
  const int b = bh / a.H;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave & 1;                         // query block
  const int kw = wave >> 1;                        // key block
  const int lane = tid & 63;
  const int hl = lane >> 5;
  const int ln = lane & 31;
  const int qrow = qt * kT + qw * 32 + ln;
  const bool qvalid = qrow < a.L;

  // Q^T as the B operand: lane holds query ln, dims 16*ks + 8*hl .. +8.
  bf16x8 qf[8];
  {
    const uint16_t* qp = a.q + ((size_t(b) * a.L + (qvalid ? qrow : 0)) * a.H + h) * kD + 8 * hl;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      uint4 u = make_uint4(0, 0, 0, 0);
      if (qvalid) u = *reinterpret_cast<const uint4*>(qp + 16 * ks);
      qf[ks] = as_bf16x8(u);
    }
  }
  const uint32_t lds0 = lds_addr(&sbuf[0][0]);
  uint32_t rk[4], rv[2];                           // K rows 32 kw + ln; V^T rows ln, keys 32 kw + 16 step ..
#pragma unroll
  for (int j = 0; j < 4; ++j)
    rk[j] = lds0 + uint32_t(4096 * kw + 128 * ln + 16 * ((2 * j + hl) ^ swz(ln & 15)));
#pragma unroll
  for (int s = 0; s < 2; ++s)
    rv[s] = lds0 + 2 * kBuf + uint32_t(128 * ln + 16 * ((4 * kw + 2 * s + hl) ^ swz(ln & 15)));
  // Copies: copy t of wave w for K fills block t/2, rows 8 (w + 4 (t%2)) + lane/8;
  // for V^T rows 8 (w + 4t) + lane/8.
  const uint32_t chunk = uint32_t(16 * ((lane & 7) ^ swz(8 * (wave & 1) + (lane >> 3))));
  const uint32_t koff = uint32_t((lane >> 3) * 256) + chunk, voff = uint32_t((lane >> 3) * 128) + chunk;

  const size_t pbytes = page_bytes(kT, kD);
  const uint8_t* head_pages = uniform_ptr(a.pool + (size_t(b) * a.H + h) * a.NT * pbytes);
  const size_t slot_stride = size_t(a.B) * a.H * a.NT * pbytes;
  const int total = ((const const_i32*)a.counts)[row];
  const int first = partial ? int(int64_t(part) * total / a.split) : 0;
  const int count = partial ? int(int64_t(part + 1) * total / a.split) - first : total;
  const int32_t* list = a.idx + size_t(row) * a.nk_cap + first;
  const float c2 = a.scale_log2;

  f32x16 o[4];                                     // O^T [4 x 32 dims][32 queries]
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) o[mb] = f32x16{};
  float m = -INFINITY;                             // offset (base-2 units), -inf until the lane's first valid key
  float moff = 0.f;                                // m, or 0 while m is -inf
  float l = 0.f;                                   // this lane's share of the row sum
  float bound = -1.f;                              // row sum that raises the offset: any on the first kExact tiles

  struct Unit {
    const uint8_t* page;
    int valid;
  };
  auto unit = [&](uint32_t j) {
    const int pos = div_nt(j, a.nt_div);
    const int t = int(j) - pos * a.NT;
    return Unit{head_pages + size_t(a.slot_of[pos]) * slot_stride + size_t(t) * pbytes,
                tile_valid(a.tv, t, a.NT, a.tail, kT)};
  };
  auto copy_k = [&](const Unit& u, uint32_t buf, int t) {
    dma16(u.page + (t >> 1) * 128 + uint32_t(8 * (wave + 4 * (t & 1))) * 256u, koff,
          lds0 + buf * kBuf + uint32_t(wave) * 1024u + uint32_t(t) * 4096u);
  };
  auto copy_v = [&](const Unit& u, int t) {
    dma16(u.page + kT * kD * 2 + uint32_t(wave + 4 * t) * 1024u, voff,
          lds0 + 2 * kBuf + uint32_t(wave) * 1024u + uint32_t(t) * 4096u);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

  // One tile, its K landed: S, the weights, then (V landed) PV.
  auto tile = [&](const Unit& cur, const Unit& next, uint32_t nbuf) {
    bf16x8 x[8], p[2];
    f32x16 s = f32x16{};
#pragma unroll
    for (int t = 0; t < 4; ++t) copy_v(cur, t);
#pragma unroll
    for (int ks = 0; ks < kAhead; ++ks) x[ks] = lds_operand(rk[ks & 3] + uint32_t((ks >> 2) * 8192));
    fence();
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[ks], qf[ks], s, 0, 0, 0);
      if (ks + kAhead < 8) x[ks + kAhead] = lds_operand(rk[(ks + kAhead) & 3] + uint32_t(((ks + kAhead) >> 2) * 8192));
      if (ks & 1) copy_k(next, nbuf, ks >> 1);
      fence();
    }
    if (cur.valid < kT) {                          // padding keys of the tile never count
      int h4 = 4 * hl;
      asm volatile("" : "+v"(h4));
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (kw * 32 + 8 * (e >> 2) + h4 + (e & 3) >= cur.valid) s[e] = -INFINITY;
    }
    auto weights = [&] {
      const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
      float rs = 0.f;
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float w0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c2, -moff));
        const float w1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e + 1], c2, -moff));
        const bf16x2 w = {(__bf16)w0, (__bf16)w1};
        p[e >> 3][e & 7] = w[0];
        p[e >> 3][(e & 7) + 1] = w[1];
        rs = __builtin_amdgcn_fdot2_f32_bf16(w, ones, rs, false);
      }
      // the packed weights are formed here: the rescale that may follow rewrites
      // them, and the fp32 values would otherwise be kept for it
      asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(rs));
      return rs;
    };
    float rs = weights();
    // wave-uniform: some lane has no offset yet, or its weights sum to more than the bound
    if (__ballot(!(m > -INFINITY) || rs > bound) != 0) {
      float mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[e]);
      mx = pair_max(mx * c2);                      // c2 > 0
      const bool had = m > -INFINITY;
      const float sh = had ? fmaxf(mx - m, 0.f) : 0.f;
      const float alpha = __builtin_amdgcn_exp2f(-sh);
      m = had ? m + sh : mx;
      l *= alpha;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) o[mb] *= alpha;
      moff = (m > -INFINITY) ? m : 0.f;
      rs = weights();
    }
    l += rs;
    meet<4>();                                     // V has landed; K of the next tile may be in flight
    auto operand = [&](int i) { return lds_operand(rv[i >> 2] + uint32_t(4096 * (i & 3))); };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) x[i] = operand(i);
    fence();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i], p[i >> 2], o[i & 3], 0, 0, 0);
      if (i + kAhead < 8) x[i + kAhead] = operand(i + kAhead);
      fence();
    }
  };

  for (int base = 0; base == 0 || base < count; base += kList) {
    // the tiles of the next kList entries; entries naming a tile outside the
    // window (stale lists) count no key
    if (base > 0) meet<0>();                       // the table is no longer read
    if (wave == 0) {
      int cnt = 0;
      const int end = min(count, base + kList), cap = a.nk_cap - first;
      for (int e0 = base; e0 == 0 || e0 < end; e0 += 256) {
        uint32_t jj[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {              // (within the row, so that the count is not waited for)
          const int e = e0 + 64 * k + lane;
          jj[k] = e < cap ? uint32_t(list[e]) : 0xffffffffu;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t j = e0 + 64 * k + lane < end ? jj[k] : 0xffffffffu;
          const bool on = j < uint32_t(a.nk) && tile_valid(a.tv, int(j % uint32_t(a.NT)), a.NT, a.tail, kT) > 0;
          const uint64_t bal = __ballot(on);
          if (on) sunit[cnt + __popcll(bal & ((uint64_t(1) << lane) - 1))] = j;
          cnt += __popcll(bal);
        }
      }
      if (lane == 0) sunit[kList] = uint32_t(cnt);
    }
    meet<0>();
    const int U = __builtin_amdgcn_readfirstlane(sunit[kList]);
    if (U == 0) continue;
    auto entry = [&](int u) { return uint32_t(__builtin_amdgcn_readfirstlane(sunit[min(u, U - 1)])); };
    Unit cur = unit(entry(0)), next = unit(entry(1));
#pragma unroll
    for (int t = 0; t < 4; ++t) copy_k(cur, 0, t);
    for (int u = 0; u < U; ++u) {
      meet<0>();                                   // K of tile u has landed; its next buffer and V's are free
      const uint32_t x2 = sunit[min(u + 2, U - 1)];
      tile(cur, next, uint32_t(u + 1) & 1u);       // past the end the last K is copied again, and not read
      if (u == kExact - 1) bound = kSumBound;
      const uint32_t d = (u & 1) ? uint32_t(-int(kBuf)) : kBuf;
#pragma unroll
      for (int j = 0; j < 4; ++j) rk[j] += d;
      cur = next;
      next = unit(__builtin_amdgcn_readfirstlane(x2));
    }
    if (U & 1) {                                   // the next entries start in buffer 0 again
#pragma unroll
      for (int j = 0; j < 4; ++j) rk[j] -= kBuf;
    }
  }

  // ---- merge the two key blocks: block 1 hands (m, l, O) to block 0 ----
  l = pair_sum(l);
  meet<0>();                                       // every copy and operand read is done
  float* xo = reinterpret_cast<float*>(&sbuf[0][0]);   // [2 query blocks][4][16][64 lanes], then m and l
  float* xm = xo + 2 * 4 * 16 * 64;
  if (kw != 0) {
    xm[qw * 128 + lane] = m;
    xm[qw * 128 + 64 + lane] = l;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) xo[((qw * 4 + mb) * 16 + e) * 64 + lane] = o[mb][e];
  }
  meet<0>();
  if (kw != 0) return;
  const float m1 = xm[qw * 128 + lane], l1 = xm[qw * 128 + 64 + lane];
  const float mm = fmaxf(m, m1);
  const float f0 = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mm);
  const float f1 = (m1 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m1 - mm);
  const float lt = l * f0 + l1 * f1;
  auto merged = [&](int mb, int e) { return o[mb][e] * f0 + xo[((qw * 4 + mb) * 16 + e) * 64 + lane] * f1; };

  if (SPLIT && partial) {
    // partial: O relative to the offset mm and the row sum
    if (qvalid) {
      const size_t wrow = size_t(row - a.split_from) * a.split + part;
      float* op = a.work + (wrow * kT + qw * 32 + ln) * kD;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d0 = mb * 32 + 8 * i + 4 * hl;
          *reinterpret_cast<float4*>(op + d0) = make_float4(merged(mb, 4 * i), merged(mb, 4 * i + 1),
                                                            merged(mb, 4 * i + 2), merged(mb, 4 * i + 3));
        }
      if (hl == 0) {
        const size_t wrows = (size_t(a.B) * a.H * a.NT - a.split_from) * a.split;
        float2* ml = reinterpret_cast<float2*>(a.work + wrows * kT * kD);
        ml[wrow * kT + qw * 32 + ln] = make_float2(mm, lt);
      }
    }
    return;
  }
  if (qvalid) {
    const float inv = (lt > 0.f) ? 1.f / lt : 0.f;
    uint16_t* op = a.o + ((size_t(b) * a.L + qrow) * a.H + h) * kD;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int d0 = mb * 32 + 8 * i + 4 * hl;
        uint2 u;
        u.x = pack_bf16x2(merged(mb, 4 * i + 0) * inv, merged(mb, 4 * i + 1) * inv);
        u.y = pack_bf16x2(merged(mb, 4 * i + 2) * inv, merged(mb, 4 * i + 3) * inv);
        *reinterpret_cast<uint2*>(op + d0) = u;
      }
    if (a.lse != nullptr && hl == 0)
      a.lse[(size_t(b) * a.H + h) * a.L + qrow] = (lt > 0.f) ? (mm + log2f(lt)) * 0.69314718055994531f : -INFINITY;
  }
}

}  // namespace

hipError_t launch_attn_fwd_t64(const AttnArgs& a, hipStream_t stream) {
  const unsigned blocks = unsigned(a.B) * unsigned(a.H) * unsigned(a.NT);
  attn_fwd_kernel<false><<<blocks, 256, 0, stream>>>(a);
  return hipGetLastError();
}

hipError_t launch_attn_fwd_t64_split(const AttnArgs& a, hipStream_t stream) {
  const unsigned rows = unsigned(a.B) * unsigned(a.H) * unsigned(a.NT);
  const unsigned blocks = unsigned(a.split_from) + (rows - unsigned(a.split_from)) * unsigned(a.split);
  attn_fwd_kernel<true><<<blocks, 256, 0, stream>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_attn_split_merge(a, stream);
}

}  // namespace uf
