// Combine split-KV partials by their log-sum-exp.
//
// When the keys of a chunk are cut into disjoint ranges, range r yields the
// normalised partial o_r and lse_r.  The full result is
//   lse = log(sum_r exp(lse_r)),   o = sum_r exp(lse_r - lse) * o_r,
// the same combination the paper's debtor stage needs after reading part of
// its KV from its partner and part locally (Section 4.1).
//
// One wavefront produces one (row, head).  Few rows are bound by the chain of
// dependent loads, many by HBM (n_ranges (D + 1) 4 bytes read per row), so
// every load that can be is in flight at once: lane r takes range r's
// log-sum-exp, the wavefront forms all weights together, and its 64 / (D / 4)
// parts read the partials of as many ranges at a time, two batches of loads in
// flight, the first before the weights are known.  Measured, 8B heads, against
// one thread per 4 outputs that walked the ranges one after the other: 7 rows
// x 17 ranges 15.4 -> 4.0 us, 137 x 9 10.7 -> 6.3 us, 300 x 17 28.9 -> 19.0 us
// with one batch of four loads behind the weights; the second batch and the
// early start take another 0.6 to 1.9 us off calls with 16 to 128 ranges.
#include "internal.h"

#include <math.h>

namespace mocap {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Partials a lane requests at a time.  Up to kFewRows rows the loads' latency
// counts, above that more loads per lane only crowd the caches.  4 and 8
// ahead: 16 rows x 128 ranges 37.4 and 35.0 us with their attention, 224 x 32
// 17.2 and 16.6, 576 x 16 35.6 and 35.8, 4096 x 20 238 and 242.
constexpr int kLoadsMany = 4, kLoadsFew = 8;
constexpr int64_t kFewRows = 512;
constexpr int64_t kMaxGroupsX = ((int64_t)1 << 32) / kGroupThreads - 1;

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off));
  return x;
}

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

template <int D, int kLoadsAhead>
__global__ __launch_bounds__(kGroupThreads) void lse_merge_kernel(const MergeLaunch p) {
  constexpr int QUADS = D / 4;         // lanes that hold one partial row
  constexpr int PARTS = 64 / QUADS;    // ranges a wavefront reads at a time
  const int lane = threadIdx.x & 63;
  const int64_t rh = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kWavesPerGroup + (threadIdx.x >> 6);
  const int64_t L = p.chunk_len;
  if (rh >= L * p.h_q) return;         // a whole wavefront: no barrier follows
  const int head = (int)(rh % p.h_q);  // row-major over (row, head)
  const int64_t row = rh / p.h_q;
  const int64_t range_stride = L * p.h_q;
  const int quad = lane % QUADS, part = lane / QUADS;

  // Ranges are taken 64 at a time: lane r holds the log-sum-exp of range r, and
  // the partials of the next kLoadsAhead ranges of each part are requested
  // before those at hand are used, the first ones before any weight is known.
  const float* o = p.ws_o + rh * D + quad * 4;
  f32x4 next[kLoadsAhead];
  auto fetch = [&](int r0, int n, int i0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kLoadsAhead; ++j)
      next[j] = *reinterpret_cast<const f32x4*>(o + (r0 + min(i0 + j * PARTS + part, n - 1)) * range_stride * D);
  };
  auto load_lse = [&](int r) { return r < p.n_ranges ? p.ws_lse[r * range_stride + rh] : -INFINITY; };
  float lr = load_lse(lane);
  fetch(0, min(64, p.n_ranges), 0);
  float m = lr;
  for (int r = lane + 64; r < p.n_ranges; r += 64) m = fmaxf(m, load_lse(r));
  m = wave_max(m);
  float z = 0.f;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int r0 = 0; r0 < p.n_ranges; r0 += 64) {
    const int n = min(64, p.n_ranges - r0);
    if (r0 > 0) {
      lr = load_lse(r0 + lane);
      fetch(r0, n, 0);
    }
    // A range that no key of the row falls into (-inf) is left out, whatever
    // its O holds; a NaN reaches the result.
    const bool has_keys = lr != -INFINITY;
    const float w = has_keys ? expf(lr - m) : -1.f;
    z += has_keys ? w : 0.f;
    for (int i0 = 0; i0 < n; i0 += kLoadsAhead * PARTS) {
      f32x4 v[kLoadsAhead];
#pragma unroll
      for (int j = 0; j < kLoadsAhead; ++j) v[j] = next[j];
      if (i0 + kLoadsAhead * PARTS < n) fetch(r0, n, i0 + kLoadsAhead * PARTS);
#pragma unroll
      for (int j = 0; j < kLoadsAhead; ++j) {
        const int i = i0 + j * PARTS + part;
        float wi = __shfl(w, i & 63);  // every lane: the source lane takes part
        const bool used = i < n && !(wi < 0.f);
        wi = used ? wi : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(wi, used ? v[j][e] : 0.f, acc[e]);
      }
    }
  }
  z = wave_sum(z);
#pragma unroll
  for (int off = 32; off >= QUADS; off >>= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off);
  if (part != 0) return;
  const float inv = z > 0.f ? 1.f / z : 0.f;
  bf16x4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) out[e] = (__bf16)(acc[e] * inv);
  *reinterpret_cast<bf16x4*>(p.o + rh * D + quad * 4) = out;
  if (quad == 0) p.lse[head * L + row] = z == 0.f ? -INFINITY : m + logf(z);
}

}  // namespace

hipError_t launch_lse_merge(const MergeLaunch& p, int head_dim, hipStream_t stream) {
  const int64_t rows = (int64_t)p.chunk_len * p.h_q;
  // A dimension of a grid holds fewer than 2^32 threads (2^26 rows); more go
  // to its second dimension.
  const int64_t groups = (rows + kWavesPerGroup - 1) / kWavesPerGroup;
  const int64_t layers = (groups + kMaxGroupsX - 1) / kMaxGroupsX;
  const dim3 grid((unsigned)((groups + layers - 1) / layers), (unsigned)layers), block(kGroupThreads);
  const bool few = rows <= kFewRows;
  if (head_dim == 128) {
    if (few) {
      hipLaunchKernelGGL((lse_merge_kernel<128, kLoadsFew>), grid, block, 0, stream, p);
    } else {
      hipLaunchKernelGGL((lse_merge_kernel<128, kLoadsMany>), grid, block, 0, stream, p);
    }
  } else {
    if (few) {
      hipLaunchKernelGGL((lse_merge_kernel<64, kLoadsFew>), grid, block, 0, stream, p);
    } else {
      hipLaunchKernelGGL((lse_merge_kernel<64, kLoadsMany>), grid, block, 0, stream, p);
    }
  }
  return hipGetLastError();
}

}  // namespace mocap
