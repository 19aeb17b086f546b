// Attention of a chunk with few rows, or of little work, for gfx950 (CDNA4).
//
// A launch of the tiled kernel (chunk_attn.hip) spends 128 rows and a serial
// walk over its keys per workgroup; a chunk of few rows fills few of those
// rows, and one of little work is bound by the walk.  Here a workgroup owns one
// slot of 32 rows and its eight wavefronts take its keys in turn, 32 at a time,
// each with a softmax state of its own; the eight partials meet in LDS.
//
//   * Each wavefront copies its K and V straight to LDS (16 KiB of its own at
//     head_dim 128) and waits only for its own copies: no barrier until the
//     end.  The next step's K is requested as soon as this step's K fragments
//     are in registers, its V as soon as the V fragments are, so 64 to 128 KiB
//     per compute unit are always in flight.  What bounds it is the latency of
//     a copy (1.5 us per step when few workgroups run, against 0.4 us of MFMA)
//     and, with enough workgroups, HBM (62720 keys of 8 heads: 4.7 TB/s).
//     Fragments loaded straight from the pools into registers touch 32 lines
//     per instruction: 3.4 us per step.
//   * Rows, ranges, MFMA layouts and softmax bookkeeping are those of the tiled
//     kernel.
//
// Measured (calls back to back in a graph), tiled kernel in its best plan and
// this one: 46 tokens of 64/8/128 heads behind 316 keys 15.0 and 8.9 us, 200 of
// 32/8/128 behind 1000 22.0 and 14.6, 256 of 32/8/128 behind 2048 27 and 22,
// 10 of 16/2/64 behind 23040 25 and 13; the other way round for 64 or more
// tokens behind long prefixes (137 of 32/8/128 behind 30720: 92 and 133 us),
// where the shared tiles of the other kernel need a quarter of the traffic.
#include "attn_device.h"

namespace mocap {
namespace {

constexpr int kStepKeys = 32;  // keys a wavefront takes at a time

// The compiler may not move LDS reads across these, and the copies it does not
// count as LDS writes of its own are complete (or the reads done) behind them.
template <int N>
__device__ __forceinline__ void wait_copies() {
  asm volatile("" ::: "memory");
  wait_vmem<N>();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void drain_lds_reads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  asm volatile("" ::: "memory");
}

template <int D, bool TWO>
__global__ __launch_bounds__(kAttnThreads, 2) void chunk_attn_short_kernel(const AttnLaunch p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int KS = D / 16;
  constexpr int MD = D / 32;
  constexpr int K_ELEMS = kStepKeys * D;
  constexpr int COPIES = K_ELEMS / 8 / 64;  // 1 KiB copies of a step's K (or V)
  // Each wavefront's own K and V of one step; its partial O at the end.
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kAttnWaves][2 * K_ELEMS];
  __shared__ float part_m[kAttnWaves][kAttnWaveRows], part_l[kAttnWaves][kAttnWaveRows],
      part_f[kAttnWaves][kAttnWaveRows];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  const int l32 = lane & 31;
  const int P = p.prefix_len;
  const int L = p.chunk_len;

  // Within a KV head: range, then 32-row slot, the one with the most keys first.
  const int logical = xcd_contiguous(blockIdx.x, p.total_wgs);
  const int per_kv = p.pairs * p.n_ranges;
  const int kv_head = logical / per_kv;
  const int in_kv = logical - kv_head * per_kv;
  const int range = in_kv / p.pairs;
  const RowPos rows = slot_start(p, p.pairs - 1 - (in_kv - range * p.pairs));
  const int last_token = min(L - 1, rows.token + (int)div_group(p, rows.head + kAttnWaveRows - 1));
  int lo, hi;
  range_bounds(p, range, &lo, &hi);

  // Steps of this workgroup: wavefront w takes w, w + 8, ...
  const int step0 = lo / kStepKeys;
  const int steps = max(0, (min(hi, P + last_token + 1) + kStepKeys - 1) / kStepKeys - step0);
  const int begin = step0 + wave, end = step0 + steps;
  const int full_end = min(hi, P + rows.token + 1);  // keys every row sees

  const int lane_x = rows.head + l32;
  const int lane_t = (int)div_group(p, lane_x);
  const int token = rows.token + lane_t;
  const int head = kv_head * p.group + lane_x - lane_t * p.group;

  // The 32 keys of step i: K rows and V columns of one block.
  const int64_t head_stride = (int64_t)D * p.block_size;
  struct Source {
    __amdgpu_buffer_rsrc_t k, v;
  };
  auto locate = [&](int i) __attribute__((always_inline)) {
    const int pos = i * kStepKeys;
    const int t = pos / kTileKeys;
    const bool remote = TWO && t >= p.remote_begin && t < p.remote_end;
    const const_i32_ptr table = (const_i32_ptr)(remote ? p.table_r : p.table);
    const int lb = (int)((__umulhi((uint32_t)pos, p.block_magic) + (uint32_t)pos) >> p.block_shift);
    const int slot = pos - lb * p.block_size;
    const int64_t base = ((int64_t)table[lb] * p.h_kv + kv_head) * head_stride;
    const uint16_t* k = (remote ? p.k_pool_r : p.k_pool) + base + (int64_t)slot * D;
    const uint16_t* v = (remote ? p.v_pool_r : p.v_pool) + base + slot;
    return Source{__builtin_amdgcn_make_buffer_rsrc((void*)k, 0, -1, kBufferWord3),
                  __builtin_amdgcn_make_buffer_rsrc((void*)v, 0, -1, kBufferWord3)};
  };
  // Copy j moves 16-byte chunks 64 j + lane of the step's K rows [32][D] and V
  // rows [D][32] to the same place in LDS, from a column XORed with the row:
  // K chunk c of row r lies at c ^ (r % 16) (D = 128) or c ^ (r / 2 % 8)
  // (D = 64), V chunk c of dim row e at c ^ (e / 4 % 4), so the 16 lanes that a
  // ds_read_b128 serves at a time hit 16 different 16-byte bank groups.  The
  // rows of copy j shift the K column by 4 j chunks (mod a row), the V rows by
  // none.
  uint16_t* const kl = ring[wave];
  uint16_t* const vl = kl + K_ELEMS;
  constexpr int ROW_CHUNKS = D / 8;
  auto k_swizzle = [](int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
  const int k_copy = (lane / ROW_CHUNKS * D + ((lane % ROW_CHUNKS) ^ k_swizzle(lane / ROW_CHUNKS)) * 8) * 2;
  const int v_copy = (lane / 4 * p.block_size + ((lane & 3) ^ (lane >> 4)) * 8) * 2;
  // Before a copy the reads of the buffer it fills have returned.
  auto copy_k = [&](const Source& s) __attribute__((always_inline)) {
    drain_lds_reads();
#pragma unroll
    for (int j = 0; j < COPIES; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(s.k, (lds_ptr_t)(kl + j * 512), 16, k_copy ^ ((4 * j) % ROW_CHUNKS * 16),
                                               j * 1024, 0, 0);
  };
  auto copy_v = [&](const Source& s) __attribute__((always_inline)) {
    drain_lds_reads();
#pragma unroll
    for (int j = 0; j < COPIES; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(s.v, (lds_ptr_t)(vl + j * 512), 16, v_copy, j * 16 * p.block_size * 2, 0,
                                               0);
  };
  // Operand fragments: lane l takes row l % 32 (a key row in MFMA order, or a
  // head dim), 16 bytes of each 32.
  const int kr = key_row_order(l32);
  bf16x8 qf[KS], kf[KS], vf[2][MD];
  auto read_k = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      kf[ks] = *reinterpret_cast<const bf16x8*>(kl + kr * D + (((ks * 2 + half) ^ k_swizzle(kr)) << 3));
  };
  auto read_v = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int md = 0; md < MD; ++md)
        vf[kk][md] = *reinterpret_cast<const bf16x8*>(vl + (md * 32 + l32) * kStepKeys +
                                                      (((kk * 2 + half) ^ (l32 >> 2 & 3)) << 3));
  };

  f32x16 oacc[MD];
#pragma unroll
  for (int md = 0; md < MD; ++md) oacc[md] = f32x16{};
  // Bookkeeping as in the tiled kernel: a reference exponent fixed by the first
  // step with a visible key, l_run the sum of the bf16 probabilities, f_run
  // that of the fp32 exponentials.
  float m_run = -INFINITY, l_run = 0.f, f_run = 0.f;
  const float sl2 = p.scale_log2;

  if (begin < end) {
    const Source first = locate(begin);
    copy_k(first);
    // Lanes past the last row take that of its token; nothing of theirs is stored.
    const uint16_t* qrow = p.q + ((int64_t)min(token, L - 1) * p.h_q + head) * D + half * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
    copy_v(first);
    for (int i = begin; i < end; i += kAttnWaves) {
      const bool more = i + kAttnWaves < end;
      const Source next = locate(more ? i + kAttnWaves : i);
      // In flight, oldest first: this step's K, then its V (and in the first
      // step the row of Q, which its use waits for).
      wait_copies<COPIES>();
      read_k();
      if (more) copy_k(next);
      f32x16 s = f32x16{};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
      const int key0 = i * kStepKeys;
      if (key0 < lo || key0 + kStepKeys > full_end) {
        // This lane's scores belong to keys key0 + half * 8 + {0..7, 16..23}.
        const int a = lo - key0 - half * 8, b = min(hi, P + token + 1) - key0 - half * 8;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int key = j < 8 ? j : j + 8;
          s[j] = key >= a && key < b ? s[j] : -INFINITY;
        }
      }
      uint32_t pk[8];
      float rs, fs;
      auto probs = [&](float neg_m) __attribute__((always_inline)) {
        rs = fs = 0.f;
#pragma unroll
        for (int j = 0; j < 16; j += 2) {
          const float e0 = __builtin_amdgcn_exp2f(fmaf(s[j], sl2, neg_m));
          const float e1 = __builtin_amdgcn_exp2f(fmaf(s[j + 1], sl2, neg_m));
          pk[j / 2] = pack_bf16x2(e0, e1);
          fs += e0 + e1;
          rs = dot2_bf16(pk[j / 2], 0x3F803F80u, rs);
        }
      };
      probs(-m_run);
      const bool over = !(rs <= kSumLimit);
      if (__builtin_amdgcn_ballot_w64(over) != 0) {
        const bool row_over = lane_pair_max(over ? 1.f : 0.f) > 0.f;
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < 16; ++j) mx = fmaxf(mx, s[j]);
        mx = lane_pair_max(mx) * sl2;
        if (row_over) {
          if (lane_pair_sum(l_run) != 0.f) {
            const float f = __builtin_amdgcn_exp2f(m_run - mx);
#pragma unroll
            for (int md = 0; md < MD; ++md) oacc[md] *= f;
            l_run *= f;
            f_run *= f;
          }
          m_run = mx;
          probs(m_run == -INFINITY ? 0.f : -m_run);
        }
      }
      l_run += rs;
      f_run += fs;
      if (more) {
        wait_copies<COPIES>();  // all but the next step's K
      } else {
        wait_copies<0>();
      }
      read_v();
      if (more) copy_v(next);
      if (key0 + kStepKeys > P + L) {
        // Unwritten store memory may hold NaN; its probabilities are 0.
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int valid = P + L - key0 - kk * 16 - half * 8;  // of this lane's 8 keys
#pragma unroll
          for (int md = 0; md < MD; ++md) {
            u32x4 w = __builtin_bit_cast(u32x4, vf[kk][md]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              w[e] &= valid > 2 * e + 1 ? 0xFFFFFFFFu : valid > 2 * e ? 0x0000FFFFu : 0u;
            vf[kk][md] = __builtin_bit_cast(bf16x8, w);
          }
        }
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pk[kk * 4], pk[kk * 4 + 1], pk[kk * 4 + 2], pk[kk * 4 + 3]});
#pragma unroll
        for (int md = 0; md < MD; ++md)
          oacc[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kk][md], pb, oacc[md], 0, 0, 0);
      }
    }
  }

  // Partials of the wavefronts meet in LDS.  A wavefront without steps leaves
  // a sum of 0, so its weight is 0 and its O is not read.
  const float l_tot = lane_pair_sum(l_run), f_tot = lane_pair_sum(f_run);
  if (half == 0) {
    part_m[wave][l32] = m_run;
    part_l[wave][l32] = l_tot;
    part_f[wave][l32] = f_tot;
  }
  if (begin < end) {
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        reinterpret_cast<f32x4*>(ring[wave])[(md * 4 + j) * 64 + lane] =
            f32x4{oacc[md][j * 4], oacc[md][j * 4 + 1], oacc[md][j * 4 + 2], oacc[md][j * 4 + 3]};
  }
  __syncthreads();

  // Wavefront w sums the pieces (md, j) = w, w + 8, ... of all partials; the
  // row of a lane stays the same.  A partial counts if its sum is not 0: a NaN
  // score leaves m = -inf (fmaxf drops it) and a NaN sum, which has to reach
  // O and the log-sum-exp.
  float m = -INFINITY;
#pragma unroll
  for (int w = 0; w < kAttnWaves; ++w) m = fmaxf(m, part_m[w][l32]);
  float weight[kAttnWaves], l = 0.f, f = 0.f;
  bool counts[kAttnWaves];
#pragma unroll
  for (int w = 0; w < kAttnWaves; ++w) {
    const float l_w = part_l[w][l32];
    counts[w] = l_w != 0.f;
    weight[w] = counts[w] ? __builtin_amdgcn_exp2f(part_m[w][l32] - m) : 0.f;
    l += l_w * weight[w];
    f += part_f[w][l32] * weight[w];
  }
  if (token >= L) return;
  const float inv = l > 0.f ? 1.f / l : 0.f;
  const float row_lse = f == 0.f ? -INFINITY : (m + log2f(f)) * kLn2;
  const bool split = p.n_ranges > 1;
  const int64_t out_row = (int64_t)token * p.h_q + head;
  const int64_t ws_row = (int64_t)range * L * p.h_q + out_row;
#pragma unroll
  for (int piece = wave; piece < MD * 4; piece += kAttnWaves) {
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kAttnWaves; ++w) {
      const f32x4 o_w = reinterpret_cast<const f32x4*>(ring[w])[piece * 64 + lane];
      // The ring of a wavefront without steps holds anything.
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] += weight[w] * (counts[w] ? o_w[e] : 0.f);
    }
    o *= inv;
    const int dim = piece * 8 + half * 4;  // (md, j) covers dims md * 32 + j * 8
    if (!split) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (__bf16)o[e];
      *reinterpret_cast<bf16x4*>(p.o + out_row * D + dim) = v;
    } else {
      *reinterpret_cast<f32x4*>(p.ws_o + ws_row * D + dim) = o;
    }
  }
  if (wave == 0 && half == 0) {
    if (split) {
      p.ws_lse[ws_row] = row_lse;
    } else {
      p.lse[(int64_t)head * L + token] = row_lse;
    }
  }
#endif  // __HIP_DEVICE_COMPILE__
}

template <int D>
void launch(const AttnLaunch& p, hipStream_t stream) {
  const dim3 grid(p.total_wgs), block(kAttnThreads);
  if (p.remote_end > p.remote_begin) {
    hipLaunchKernelGGL((chunk_attn_short_kernel<D, true>), grid, block, 0, stream, p);
  } else {
    hipLaunchKernelGGL((chunk_attn_short_kernel<D, false>), grid, block, 0, stream, p);
  }
}

}  // namespace

hipError_t launch_chunk_attn_short(const AttnLaunch& p, int head_dim, hipStream_t stream) {
  if (head_dim == 128) {
    launch<128>(p, stream);
  } else {
    launch<64>(p, stream);
  }
  return hipGetLastError();
}

}  // namespace mocap
