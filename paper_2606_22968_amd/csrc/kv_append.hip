// Append one chunk's keys/values to the block-addressed KV store.
//
// Each chunk produces new KV that later chunks keep reading (Section 2.2);
// under the paper's memory-balanced reallocation (Section 4.1) a stage first
// produces the chunk's KV and then places it, locally or at its partner, so
// the store is addressed through a block table.  This kernel is a pure
// bit copy:
//   K: [L][Hkv][D] -> k_pool[phys][h][slot][:]        (row per position)
//   V: [L][Hkv][D] -> v_pool[phys][h][:][slot]        (transposed per block)
// with phys = table[(P + t) / bs] and slot = (P + t) % bs.
//
// The kernel is bound by HBM (8 * len * Hkv * D bytes) and, below a few
// thousand positions, by latency.  One workgroup moves the positions of one
// KV head that fall into one 64-slot tile of the store, aligned to the tile:
// wherever a chunk starts, only its first and last tile are partial, one block
// holds the whole tile, and V leaves in whole 128-byte lines (64 slots of one
// head-dim row).  Tiles counted from the chunk's start instead left every tile
// of a chunk that starts off the grid to 2-byte stores.  Measured (kernel
// time, inputs not in cache): 20011 positions from 8191, 8 heads of 128:
// 53.9 -> 36.1 us (3.0 -> 4.5 TB/s; a large device copy reaches 5.2); 2048
// positions on the grid: 5.0 -> 5.1 us (tiles of 32 positions: 38.1 and
// 5.0 us; half or a quarter of the threads with more loads each: 36 and
// 5.2-7.1 us).
//
// One 16-byte chunk of K and one of V per thread (D / 8 threads per position).
// Each thread issues both loads first (the pools may alias nothing the loads
// read, but the compiler cannot know that, so a load placed after a store
// would wait for it), writes its K chunk out as one 16-byte store and scatters
// its V chunk into an LDS tile [D][64 positions].  After one barrier the tile
// leaves as 16-byte stores of 8 consecutive slots of one head-dim row, or
// 2-byte stores where a group of 8 slots is not all the chunk's.
//
// LDS tile: 16-byte chunk (e, q) holds positions 8q .. 8q+7 of dim e and is
// stored at chunk slot (8 e + q) ^ ((e / 8) % 16).  For D = 128 a 2-byte
// write instruction (16 chunk columns ch, dims e = 8 ch + k, positions
// t, t+2, t+4, t+6) then lands in 16 distinct groups of four banks, one
// dword of each bank, and the 16 lanes that a 16-byte read serves at a time
// (dims e and e + 1 with e even, all q) stay in distinct groups too: no bank
// conflicts.  (D = 64 has 8 chunk columns and writes two lanes per bank.)
#include "internal.h"

namespace mocap {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kAppendTokens = 64;  // slots per workgroup, aligned (divides every block size)

template <int D>
constexpr int append_threads() { return kAppendTokens * (D / 8); }

// Element index of (dim e, position tok) in the tile.
__device__ __forceinline__ int v_index(int e, int tok) {
  return (((e * (kAppendTokens / 8) + (tok >> 3)) ^ ((e >> 3) & 15)) << 3) + (tok & 7);
}

template <int D>
__global__ __launch_bounds__(append_threads<D>()) void kv_append_kernel(const AppendLaunch p) {
  constexpr int T = kAppendTokens;
  constexpr int ROW_CHUNKS = D / 8;  // 16-byte chunks per position
  __shared__ __attribute__((aligned(16))) uint16_t vt[D * T];

  const int tid = threadIdx.x;
  const int h = blockIdx.y;
  // Absolute positions [tile0, tile0 + T) with tile0 a multiple of T: one
  // block holds them (block_size is a multiple of 64).  Tile slots
  // [first, last) belong to the chunk.
  const int64_t tile0 = (p.start_pos / T + blockIdx.x) * T;
  const int first = (int)max(p.start_pos - tile0, (int64_t)0);
  const int last = (int)min(p.start_pos + p.chunk_len - tile0, (int64_t)T);
  const uint32_t lb = (uint32_t)tile0 / (uint32_t)p.block_size;
  const int64_t slot0 = tile0 - (int64_t)lb * p.block_size;
  const int64_t head_row = (int64_t)p.table[lb] * p.h_kv + h;

  // Thread -> (position, chunk): the D / 8 lanes of a position read its
  // whole K and V rows, consecutive 16-byte pieces.  A wavefront takes every
  // other position of 2 * PW consecutive ones (wave pairs share them), so its
  // 2-byte tile writes cover all four dwords of each 16-byte chunk.
  constexpr int PW = 64 / ROW_CHUNKS;  // positions per wavefront
  const int wv = tid >> 6, wl = tid & 63;
  const int tok = (wv >> 1) * 2 * PW + (wv & 1) + 2 * (wl / ROW_CHUNKS), ch = wl % ROW_CHUNKS;
  if (tok >= first && tok < last) {
    const int64_t src = ((tile0 + tok - p.start_pos) * p.h_kv + h) * D + ch * 8;
    const u32x4 kr = *reinterpret_cast<const u32x4*>(p.k_chunk + src);
    const u32x4 vr = *reinterpret_cast<const u32x4*>(p.v_chunk + src);
    *reinterpret_cast<u32x4*>(p.k_pool + (head_row * p.block_size + slot0 + tok) * D + ch * 8) = kr;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int e = ch * 8 + 2 * w;
      vt[v_index(e, tok)] = (uint16_t)(vr[w] & 0xFFFFu);
      vt[v_index(e + 1, tok)] = (uint16_t)(vr[w] >> 16);
    }
  }
  __syncthreads();

  // Thread -> (dim row e, group of 8 slots).
  const int e = tid / (T / 8), slot = tid % (T / 8) * 8;
  uint16_t* dst = p.v_pool + (head_row * D + e) * p.block_size + slot0 + slot;
  const uint16_t* tile = vt + v_index(e, slot);
  if (slot >= first && slot + 8 <= last) {
    *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(tile);
  } else {
    for (int j = max(first - slot, 0); j < min(last - slot, 8); ++j) dst[j] = tile[j];
  }
}

}  // namespace

hipError_t launch_kv_append(const AppendLaunch& p, int head_dim, hipStream_t stream) {
  const int64_t first_tile = p.start_pos / kAppendTokens;
  const int64_t end_tile = (p.start_pos + p.chunk_len + kAppendTokens - 1) / kAppendTokens;
  const dim3 grid((unsigned)(end_tile - first_tile), p.h_kv);
  if (head_dim == 128) {
    hipLaunchKernelGGL(kv_append_kernel<128>, grid, dim3(append_threads<128>()), 0, stream, p);
  } else {
    hipLaunchKernelGGL(kv_append_kernel<64>, grid, dim3(append_threads<64>()), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace mocap
