// Device helpers shared by the attention kernels (gfx950).
#pragma once

#include "../launch.h"
#include "../xcd_order.h"

namespace uf {
namespace attn {

constexpr int kD = 128;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(4))) int32_t const_i32;   // uniform -> scalar loads

__device__ inline bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// Both lanes of a pair (l, l^32) get the same value.
__device__ inline float pair_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// One 16-byte-per-lane copy global -> LDS: lane l reads base + off and writes
// LDS byte lds + 16*l.  Issued as inline assembly so that the compiler's
// wait-count insertion does not treat every later LDS read as dependent on it;
// the kernels order the copies with explicit s_waitcnt vmcnt and barriers.
// The uniform base is a scalar pair and the LDS target goes through m0.
__device__ inline void dma16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds) : "memory");
}

// j / NT for 0 <= j < 2^31 from d = (2^64 - 1) / NT: ((j + 1) * d) >> 64 in
// scalar integer arithmetic (a division by a run-time value would otherwise
// use vector float instructions in the softmax waves).  With d = (2^64 - r) / NT,
// 0 < r <= NT, the product is (j + 1) / NT minus less than 2^-32, which floors
// to j / NT.
__device__ __forceinline__ int div_nt(uint32_t j, uint64_t d) {
  const uint64_t x = uint64_t(j) + 1u;
  const uint64_t lo = x * uint32_t(d);
  const uint64_t hi = x * uint32_t(d >> 32);
  return int((hi + (lo >> 32)) >> 32);
}

// A pointer that is the same on every lane, held in scalar registers.
__device__ __forceinline__ const uint8_t* uniform_ptr(const uint8_t* q) {
  const uint64_t p = reinterpret_cast<uint64_t>(q);
  // (the builtin returns int: widen through uint32_t, not by sign extension)
  const uint64_t lo = uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(p)));
  const uint64_t hi = uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(p >> 32)));
  return reinterpret_cast<const uint8_t*>(lo | (hi << 32));
}

// Item of workgroup i in a launch (or its part) whose items 0 .. whole-1 are whole rows
// and the n - whole others slices of rows whole .. rows-1; the launch has `items`.
// Contiguous ranges per XCD where heads are short enough for that to pay and no
// XCD gets much more to do by it (xcd_order.h).  With no more items than CUs every
// one has its own CU, whatever the order.
__device__ __forceinline__ int xcd_deal(int i, int n, int whole, int rows, int items, int NT, int resident,
                                        const int32_t* counts) {
  if (NT * 4 > resident) return i;
  if (items > 256) {
    const bool slice = i >= whole;
    if (!xcd_even((const const_i32*)counts + (slice ? whole : 0), slice ? rows - whole : whole)) return i;
  }
  return xcd_split_item(i, n, whole, NT, resident);
}

// s_waitcnt immediates (gfx9 encoding): vmcnt in [3:0] and [15:14], expcnt
// in [6:4], lgkmcnt in [11:8].
constexpr int waitcnt_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// s_waitcnt vmcnt(N) lgkmcnt(0), then the workgroup barrier; the signal fences
// keep the compiler from moving LDS accesses across it.
template <int N>
__device__ __forceinline__ void meet() {
  constexpr int imm = (N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(imm);
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// 3-bit XOR pattern of LDS row r (r % 16): bijective in bits 0..2 for either
// value of bit 3, and in bits 1..3 for either value of bit 0.
__device__ __forceinline__ int swz(int r) {
  const int b3 = (r >> 3) & 1;
  return ((((r >> 2) & 1) ^ b3) << 2) | (r & 2) | ((r & 1) ^ b3);
}

__device__ inline uint32_t lds_addr(const void* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void*)p);
}

}  // namespace attn
}  // namespace uf
