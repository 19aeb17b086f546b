// Internal launch descriptions shared by the host API and the HIP kernels of
// libmocap_attn.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mocap {

constexpr int kTileKeys = 64;          // keys per KV tile (LDS stage)
constexpr int kAttnWaves = 8;          // wavefronts per attention workgroup
constexpr int kAttnWaveRows = 32;      // query rows owned by one attention wavefront
constexpr int kAttnThreads = 64 * kAttnWaves;
constexpr int kWavesPerGroup = 4;      // wavefronts per workgroup of the other kernels
constexpr int kGroupThreads = 64 * kWavesPerGroup;

// One launch of the attention kernel.  The rows of a KV head are the (token,
// query head) pairs of its group in token-major order: row f is token f / G,
// head f % G.  A workgroup holds two units of four wavefronts; a unit owns 128
// consecutive rows (a row group), 32 per wavefront.  The units of a workgroup
// take two row groups for one KV range: pair q is row groups q and
// row_groups - 1 - q (mirrored; the middle group of an odd count is alone),
// row_groups - 2 - 2q and row_groups - 1 - 2q (adjacent, longest pair first;
// group 0 alone when the count is odd), or row_groups - 1 - q alone (single).
// A unit without a group of its own takes half of every tile of the other
// unit's group.
// kShort is the other attention kernel (chunk_attn_short.hip): a workgroup
// owns one slot of 32 rows and its wavefronts share the slot's keys; `pairs`
// counts those slots.
//
// KV ranges: n_ranges == 1 is the unsplit launch over [0, P + L).  Otherwise
// the span_tiles tiles of [0, span_end) are cut evenly into span_parts ranges,
// and a range n_ranges > span_parts is the chunk's own keys [P, P + L): either
// all of [0, P + L) is cut (span_parts == n_ranges), or the prefix is and the
// chunk's keys are the last range (span_parts == n_ranges - 1).  Tile t holds
// keys [64 t, 64 t + 64); tiles [remote_begin, remote_end) are read from the
// second store, every other tile from the first.
enum Pairing { kMirrored = 0, kAdjacent = 1, kSingle = 2, kShort = 3 };

struct AttnLaunch {
  const uint16_t* q;        // bf16 [L][Hq][D]
  const uint16_t* k_pool;   // bf16 [nb][Hkv][bs][D]
  const uint16_t* v_pool;   // bf16 [nb][Hkv][D][bs]
  const int32_t* table;     // logical block -> physical block
  const uint16_t* k_pool_r; // second store (same layout and block size), or null
  const uint16_t* v_pool_r;
  const int32_t* table_r;
  uint16_t* o;              // bf16 [L][Hq][D]         (unsplit)
  float* lse;               // fp32 [Hq][L]            (unsplit)
  float* ws_o;              // fp32 [R][L][Hq][D]      (split partials)
  float* ws_lse;            // fp32 [R][L][Hq]
  int32_t prefix_len;       // P (P + L < 2^31 - 128, checked on the host)
  int32_t span_tiles;       // tiles cut into ranges
  int32_t span_parts;       // ranges they are cut into
  int32_t span_end;         // end of their keys: P + L or P
  int32_t chunk_len;        // L
  int32_t h_q;
  int32_t h_kv;
  int32_t group;            // Hq / Hkv
  uint32_t group_magic;     // floor(n / group) = (umulhi(n, magic) + n) >> shift
  int32_t group_shift;      //   for 0 <= n < 2^31
  int32_t row_groups;       // ceil(L group / 128)
  int32_t pairing;          // Pairing
  int32_t pairs;            // workgroups of one KV head and range
  int32_t block_size;
  uint32_t block_magic;     // floor(n / block_size) = (umulhi(n, magic) + n) >> shift
  int32_t block_shift;      //   for 0 <= n < 2^31 (division by an invariant integer)
  int32_t n_ranges;         // 1 = unsplit
  int32_t remote_begin;     // tiles [remote_begin, remote_end) live in the second store
  int32_t remote_end;
  int32_t total_wgs;
  float scale_log2;         // scale * log2(e)
};

struct AppendLaunch {
  const uint16_t* k_chunk;  // bf16 [L][Hkv][D]
  const uint16_t* v_chunk;  // bf16 [L][Hkv][D]
  uint16_t* k_pool;
  uint16_t* v_pool;
  const int32_t* table;
  int64_t start_pos;
  int32_t chunk_len;
  int32_t h_kv;
  int32_t block_size;
};

struct MergeLaunch {
  const float* ws_o;        // fp32 [R][L][Hq][D]
  const float* ws_lse;      // fp32 [R][L][Hq]
  uint16_t* o;              // bf16 [L][Hq][D]
  float* lse;               // fp32 [Hq][L]
  int32_t chunk_len;
  int32_t h_q;
  int32_t n_ranges;
};

hipError_t launch_chunk_attn(const AttnLaunch& p, int head_dim, hipStream_t stream);
hipError_t launch_chunk_attn_short(const AttnLaunch& p, int head_dim, hipStream_t stream);
hipError_t launch_kv_append(const AppendLaunch& p, int head_dim, hipStream_t stream);
hipError_t launch_lse_merge(const MergeLaunch& p, int head_dim, hipStream_t stream);

}  // namespace mocap
