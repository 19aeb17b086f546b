// Device code shared by the two attention kernels.
#pragma once

#include "internal.h"

#include <math.h>

namespace mocap {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float lane_pair_max(float x) {
  // v_permlane32_swap exchanges the upper half of one operand with the lower
  // half of the other; the max over both results is max(x[l], x[l ^ 32]).
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float lane_pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Row order of K inside a 32-key MFMA block: bits 2 and 3 swapped.
__device__ __forceinline__ int key_row_order(int m) {
  return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

// Workgroup ids are handed to the 8 XCDs round robin.  Renumber them so each
// XCD receives one contiguous run of logical items: consecutive items share a
// KV head, so the tiles they stream stay in that XCD's L2.
__device__ __forceinline__ int xcd_contiguous(int hw_id, int n) {
  const int xcd = hw_id & 7, slot = hw_id >> 3;
  const int per = n >> 3, rem = n & 7;
  return xcd * per + min(xcd, rem) + slot;
}

// The first row of 32-row slot s of a KV head: rows are the (token, query
// head) pairs of the group in token-major order, so slot s starts at row 32 s:
// token 32 s / G, head 32 s % G of the group.
struct RowPos {
  int token, head;
};
__device__ __forceinline__ uint32_t div_group(const AttnLaunch& p, uint32_t n) {
  return (__umulhi(n, p.group_magic) + n) >> p.group_shift;
}
__device__ __forceinline__ RowPos slot_start(const AttnLaunch& p, int s) {
  const int a = (int)div_group(p, s);
  const int x = (s - a * p.group) * kAttnWaveRows;
  const int t = (int)div_group(p, x);
  return RowPos{a * kAttnWaveRows + t, x - t * p.group};
}

// Keys [lo, hi) of a KV range.
__device__ __forceinline__ void range_bounds(const AttnLaunch& p, int range, int* lo, int* hi) {
  if (p.n_ranges == 1) {
    *lo = 0;
    *hi = p.prefix_len + p.chunk_len;
  } else if (range < p.span_parts) {
    *lo = (int)((int64_t)p.span_tiles * range / p.span_parts) * kTileKeys;
    *hi = min((int)((int64_t)p.span_tiles * (range + 1) / p.span_parts) * kTileKeys, p.span_end);
  } else {
    *lo = p.prefix_len;
    *hi = p.prefix_len + p.chunk_len;
  }
}

// Softmax bookkeeping.  Each query row keeps a reference exponent m (base 2)
// and accumulates p = exp2(s * scale * log2(e) - m) without taking block
// maxima.  m is only a scale: the result sum(p v) / sum(p) does not depend on
// it as long as nothing overflows, and fp32/bf16 keep their relative
// precision over the whole exponent range.  m is fixed by the first block of
// the row that has a visible key, while nothing has been accumulated yet, so
// the O accumulator never needs rescaling.  A later block whose partial row
// sum exceeds kSumLimit = 2^60 (a score more than ~60 binary orders above the
// first block's maximum, which ordinary attention scores never reach) marks
// the row: its m is raised to that block's maximum, its O accumulator and
// row sums (all of earlier blocks, taken with the old m) are scaled by
// 2^(m_old - m_new), and the block's probabilities are recomputed before
// they reach the P*V product.  The loop itself never rescales.
constexpr float kSumLimit = 1152921504606846976.0f;  // 2^60

typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;
// Word 3 of a raw (untyped) buffer descriptor: 32-bit data format.
constexpr int kBufferWord3 = 0x00020000;

// s_waitcnt immediates in the gfx9 encoding (vmcnt in bits 3:0 and 15:14,
// expcnt in 6:4, lgkmcnt in 11:8).  Written as builtins, not inline
// assembly, so the compiler's own wait insertion knows what has completed.
constexpr int kWaitLgkm0 = 0xC07F;
template <int N>
__device__ __forceinline__ void wait_vmem() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x70 | 0xF00);
}

}  // namespace
}  // namespace mocap
