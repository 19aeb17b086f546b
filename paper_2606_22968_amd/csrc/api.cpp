// Host side of libmocap_attn's device calls: argument validation, split
// planning and kernel dispatch.  Every check runs before anything is
// enqueued.  The host-only chunk planners live in plan.cpp.
#include "mocap_attn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "internal.h"

namespace {

// Magic number and shift for unsigned division by an invariant d >= 1, valid
// for dividends below 2^31: l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1,
// and n / d = (umulhi(n, m) + n) >> l (Granlund and Montgomery, 1994, round-up
// method; the sum cannot overflow 32 bits because umulhi(n, m) <= n < 2^31).
void block_divider(uint32_t d, uint32_t* magic, int32_t* shift) {
  int l = 0;
  while ((1ull << l) < d) ++l;
  *magic = (uint32_t)((((1ull << l) - d) << 32) / d + 1);
  *shift = l;
}

using mocap::kTileKeys;
using mocap::kAttnWaveRows;
using mocap::kAttnWaves;

constexpr int kMaxDevices = 64;
constexpr int64_t kMaxPositions = ((int64_t)1 << 31) - 128;
std::atomic<int> g_cu_count[kMaxDevices];  // 0 = not yet queried

bool aligned16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0; }

bool supported_head_dim(int d) { return d == 64 || d == 128; }

mocap_status device_cu_count(int* out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MOCAP_ERR_HIP;
  if (dev >= 0 && dev < kMaxDevices) {
    const int cached = g_cu_count[dev].load(std::memory_order_relaxed);
    if (cached > 0) {
      *out = cached;
      return MOCAP_OK;
    }
  }
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    return MOCAP_ERR_HIP;
  if (dev >= 0 && dev < kMaxDevices) g_cu_count[dev].store(cus, std::memory_order_relaxed);
  *out = cus;
  return MOCAP_OK;
}

// Rows (token, query head of the KV head's group) of one unit of four waves.
constexpr int kUnitRows = kAttnWaveRows * kAttnWaves / 2;

struct Plan {
  int row_groups;
  int pairs;
  int base_wgs;      // workgroups of one KV range when row groups are paired
  int64_t units;     // size of the chunk (bounded by make_plan)
  int64_t prefix_tiles;
  int n_ranges;
  bool own_range;    // the chunk's own keys are a range of their own (requested splits)
  size_t ws_bytes;
  // Prefix tiles [remote_begin, remote_end) come from a second store.
  int64_t remote_begin = 0, remote_end = 0;
};

size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

size_t workspace_for(int n_ranges, int64_t chunk_len, int h_q, int head_dim) {
  if (n_ranges <= 1) return 0;
  const size_t rows = (size_t)n_ranges * (size_t)h_q * (size_t)chunk_len;
  return round_up(rows * (size_t)head_dim * sizeof(float), 256) + round_up(rows * sizeof(float), 256);
}

// One attention launch as the planner sees it.
struct LaunchShape {
  int64_t prefix_len;
  int32_t chunk_len, h_q, h_kv, head_dim;
  int row_groups;
  int slots;  // compute units
};

// Time model of one launch, used to choose the KV ranges and the pairing.
//   * A workgroup costs a tile time per 64-key tile that both of its units
//     compute and kLoneTile times that for a tile only its longer unit
//     computes (two waves share its rows' keys, or one wave per SIMD works),
//     plus a group time of fixed work; one workgroup per compute unit at a time
//     (the attention kernel's LDS ring fills a CU).
//   * The launch time is the makespan of the workgroups in the order the
//     hardware hands them out: each XCD takes one contiguous run of the
//     logical order and starts the next workgroup on whichever of its compute
//     units is free (so a count just above a whole number per compute unit
//     costs a second round: 39 workgroups per range on 256 compute units run
//     at 75 us in 6 ranges and 109 us in 7).  Plus, when split, the merge: a
//     launch and its traffic (the partials, written and read) at
//     kMergeBytesPerUs.
// The constants were measured on MI355X, on launches short enough that the
// clock holds; only the ranking of candidate plans depends on them.
constexpr double kTileUs128 = 1.25, kTileUs64 = 0.8;
constexpr double kGroupUs128 = 5.0, kGroupUs64 = 3.5;
constexpr double kMergeBytesPerUs = 5.0e6;
constexpr double kLaunchUs = 6.0;
// Rates at which the tiled and the short kernel stream keys and values from
// HBM (382 MB: 82 and 95 us).  They decide between the two; the weight below 1
// keeps enough ranges in a plan to reach them (102 MB: 28 us, and 36 us with
// the fewer ranges that weight 1 chooses).
constexpr double kTileBytesPerUs = 4.7e6, kShortBytesPerUs = 4.2e6;
constexpr double kStreamWeight = 0.6;
constexpr double kLoneTile = 0.65;
constexpr int kXcds = 8;
// A workgroup's row groups (see AttnLaunch): single placements are looked at
// up to this many workgroups per compute unit.
using mocap::kAdjacent;
using mocap::kMirrored;
using mocap::kShort;
using mocap::kSingle;
constexpr int64_t kSingleRounds = 2;
// The short kernel: one round of steps of a workgroup's eight wavefronts (32
// keys each), fixed work, and how many workgroups per compute unit are looked at.
constexpr double kStepUs128 = 1.5, kStepUs64 = 0.8;
constexpr double kShortGroupUs = 2.0;
constexpr int64_t kShortRounds = 4;

// Workgroups of one KV head and range.
int workgroups_of_rows(int64_t rows, int pairing) {
  const int64_t groups = (rows + kUnitRows - 1) / kUnitRows;
  return (int)(pairing == kShort    ? (rows + kAttnWaveRows - 1) / kAttnWaveRows
               : pairing == kSingle ? groups
                                    : (groups + 1) / 2);
}

// Infinity if the mean load alone reaches `limit`.
double estimate_launch_us(const LaunchShape& x, int n_ranges, bool own_range, int pairing, double limit) {
  const int group = x.h_q / x.h_kv;
  const int64_t rows = (int64_t)x.chunk_len * group;
  const int unit_rows = pairing == kShort ? kAttnWaveRows : kUnitRows;
  const int row_groups = (int)((rows + unit_rows - 1) / unit_rows);
  const int pairs = workgroups_of_rows(rows, pairing);
  const double group_us = x.head_dim == 128 ? kGroupUs128 : kGroupUs64;
  const double step_us = x.head_dim == 128 ? kStepUs128 : kStepUs64;
  const double tile_us = x.head_dim == 128 ? kTileUs128 : kTileUs64;
  const int64_t prefix_tiles = (x.prefix_len + kTileKeys - 1) / kTileKeys;
  const int64_t all_tiles = (x.prefix_len + x.chunk_len + kTileKeys - 1) / kTileKeys;
  const int parts = own_range ? n_ranges - 1 : n_ranges;
  const int64_t span = own_range ? prefix_tiles : all_tiles;
  // Tiles the unit of row group rg visits among tiles [t0, t1).
  auto unit_tiles = [&](int rg, int64_t t0, int64_t t1) -> int64_t {
    if (rg < 0) return 0;
    const int64_t tokens = std::min<int64_t>(x.chunk_len, ((int64_t)(rg + 1) * unit_rows + group - 1) / group);
    const int64_t end = (x.prefix_len + tokens + kTileKeys - 1) / kTileKeys;
    return std::max<int64_t>(0, std::min(t1, end) - t0);
  };
  std::vector<double> cost;  // of one KV head, in logical order
  cost.reserve((size_t)pairs * n_ranges);
  for (int r = 0; r < n_ranges; ++r) {
    const int64_t t0 = r < parts ? span * r / parts : x.prefix_len / kTileKeys;
    const int64_t t1 = r < parts ? span * (r + 1) / parts : all_tiles;
    for (int q = 0; q < pairs; ++q) {
      // Pair q: row groups q and R-1-q, R-2-2q and R-1-2q, or R-1-q alone.
      const int top = pairing == kAdjacent ? row_groups - 1 - 2 * q : row_groups - 1 - q;
      const int other = pairing >= kSingle ? -1 : pairing == kAdjacent ? top - 1 : q < top ? q : -1;
      const int64_t a = unit_tiles(top, t0, t1), b = unit_tiles(other, t0, t1);
      if (pairing == kShort) {
        cost.push_back((double)((2 * a + kAttnWaves - 1) / kAttnWaves) * step_us + kShortGroupUs);
      } else {
        cost.push_back(((double)std::min(a, b) + (double)(std::max(a, b) - std::min(a, b)) * kLoneTile) * tile_us +
                       group_us);
      }
    }
  }
  double fixed = kLaunchUs;
  if (n_ranges > 1) {
    const double partial = (double)n_ranges * x.chunk_len * x.h_q * (x.head_dim + 1) * 4.0;
    fixed += 2.0 * partial / kMergeBytesPerUs + kLaunchUs;
  }
  const int64_t total_wgs = (int64_t)cost.size() * x.h_kv;
  const int xcd_slots = std::max(1, x.slots / kXcds);
  double sum = 0.0;
  for (double c : cost) sum += c;
  const double mean = sum * x.h_kv / (xcd_slots * kXcds);
  if (fixed + mean >= limit) return INFINITY;
  double makespan = 0.0;
  int64_t next = 0;
  const int64_t size = (int64_t)cost.size();
  std::pair<int64_t, int64_t> seen[kXcds];  // (first workgroup of its KV head, count) of the XCDs so far
  std::vector<double> busy_until;
  for (int xcd = 0; xcd < kXcds; ++xcd) {
    const int64_t begin = next, count = total_wgs / kXcds + (xcd < total_wgs % kXcds ? 1 : 0);
    next += count;
    seen[xcd] = {begin % size, count};
    if (std::find(seen, seen + xcd, seen[xcd]) != seen + xcd) continue;  // runs the same workgroups
    busy_until.clear();
    for (int64_t i = begin; i < next; ++i) {
      double t = cost[(size_t)(i % size)];
      if ((int)busy_until.size() == xcd_slots) {
        if (i - begin == xcd_slots) std::make_heap(busy_until.begin(), busy_until.end(), std::greater<double>());
        std::pop_heap(busy_until.begin(), busy_until.end(), std::greater<double>());
        t += busy_until.back();
        busy_until.back() = t;
        std::push_heap(busy_until.begin(), busy_until.end(), std::greater<double>());
      } else {
        busy_until.push_back(t);
      }
      makespan = std::max(makespan, t);
    }
  }
  const double kv_us = 4.0 * (x.prefix_len + x.chunk_len) * x.h_kv * x.head_dim /
                       (pairing == kShort ? kShortBytesPerUs : kTileBytesPerUs);
  return fixed + std::hypot(makespan, kStreamWeight * kv_us);
}

// MOCAP_PAIRING=mirrored, =adjacent, =single or =short in the environment forces a
// pairing (for tests); -1 = choose.
int pairing_mode() {
  const char* force = std::getenv("MOCAP_PAIRING");
  if (force && std::strcmp(force, "mirrored") == 0) return kMirrored;
  if (force && std::strcmp(force, "adjacent") == 0) return kAdjacent;
  if (force && std::strcmp(force, "single") == 0) return kSingle;
  if (force && std::strcmp(force, "short") == 0) return kShort;
  return -1;
}

// The best placement of row groups in workgroups (mirrored: q with R-1-q,
// every workgroup about equally long, the units sharing the tiles only the
// longer one sees; adjacent: 2q with 2q+1, both units on their own rows nearly
// throughout, workgroups of different lengths evened out when there are many
// per compute unit; single: both units on one row group's tiles, half of each
// tile's keys, which pays where even then compute units stay free).
double best_pairing_us(const LaunchShape& x, int n_ranges, bool own_range, int* pairing_out) {
  const int mode = pairing_mode();
  int best = mode >= 0 ? mode : kMirrored;
  // In full, also where it is too long: the others are measured by it.
  double best_us = estimate_launch_us(x, n_ranges, own_range, best, INFINITY);
  if (mode < 0) {
    // Another placement only when the model expects it to win clearly.  With
    // up to two row groups the two ways to pair them are the same, with one
    // so is single.
    const int64_t rows = (int64_t)x.chunk_len * (x.h_q / x.h_kv);
    for (int pairing : {kAdjacent, kSingle, kShort}) {
      const int64_t wgs = (int64_t)workgroups_of_rows(rows, pairing) * x.h_kv * n_ranges;
      if (pairing == kAdjacent && x.row_groups <= 2) continue;
      if (pairing == kSingle && (x.row_groups <= 1 || wgs > kSingleRounds * x.slots)) continue;
      if (pairing == kShort && wgs > kShortRounds * x.slots) continue;
      const double bar = best_us * (pairing == kShort ? 0.95 : 0.98);
      const double us = estimate_launch_us(x, n_ranges, own_range, pairing, bar);
      if (us < bar) {
        best_us = us;
        best = pairing;
      }
    }
  }
  if (pairing_out) *pairing_out = best;
  return best_us;
}

struct PlanKey {
  int64_t prefix_len;
  int32_t chunk_len, h_q, h_kv, head_dim, requested, slots;
  size_t ws_cap;
  int pairing;
  bool operator==(const PlanKey& o) const {
    return prefix_len == o.prefix_len && chunk_len == o.chunk_len && h_q == o.h_q && h_kv == o.h_kv &&
           head_dim == o.head_dim && requested == o.requested && slots == o.slots && ws_cap == o.ws_cap &&
           pairing == o.pairing;
  }
};

// Small cache of automatic choices (a chunk loop asks for the same shape in
// mocap_chunk_attn_workspace_size and in mocap_chunk_attn).
std::mutex g_plan_mutex;
constexpr int kPlanCache = 64;
PlanKey g_plan_keys[kPlanCache];
int g_plan_values[kPlanCache];
int g_plan_count = 0, g_plan_next = 0;

// Most workgroups of a split launch (of few ranges, which even out the long
// chunks of a prompt, or of many, which only cost planning time beyond that),
// and fewest tiles of a range.
constexpr int64_t kSplitWgsFew = 4096, kSplitWgsMany = 2048;
constexpr int64_t kFewRanges = 8;
constexpr int64_t kMinRangeTiles = 4;

// Number of KV ranges to use.  A requested count is clamped to what the
// prefix allows (the chunk's own keys are then the last range).  0 picks the
// plan with the smallest modelled launch time among no split and even cuts of
// all keys whose workspace fits in ws_cap bytes: any count up to 16, and above
// that the counts that fill the compute units a whole number of times.
int choose_ranges(const LaunchShape& x, int base_wgs, int64_t prefix_tiles, int requested, size_t ws_cap) {
  if (prefix_tiles <= 0) return 1;
  if (requested >= 1) {
    if (requested == 1) return 1;
    const int64_t parts = requested - 1 < prefix_tiles ? requested - 1 : prefix_tiles;
    return (int)parts + 1;
  }
  const PlanKey key{x.prefix_len, x.chunk_len, x.h_q, x.h_kv, x.head_dim, requested, x.slots, ws_cap, pairing_mode()};
  {
    std::lock_guard<std::mutex> lock(g_plan_mutex);
    for (int i = 0; i < g_plan_count; ++i)
      if (g_plan_keys[i] == key) return g_plan_values[i];
  }
  int best = 1;
  // A split must pay for itself clearly.
  double best_us = 0.98 * best_pairing_us(x, 1, false, nullptr);
  auto consider = [&](int64_t n) {
    if (workspace_for((int)n, x.chunk_len, x.h_q, x.head_dim) > ws_cap) return;
    const double us = best_pairing_us(x, (int)n, false, nullptr);
    if (us < best_us) {
      best_us = us;
      best = (int)n;
    }
  };
  const int64_t all_tiles = (x.prefix_len + x.chunk_len + kTileKeys - 1) / kTileKeys;
  const int64_t max_n = std::min(all_tiles / kMinRangeTiles,
                                 std::max(std::min(kFewRanges, kSplitWgsFew / base_wgs), kSplitWgsMany / base_wgs));
  for (int64_t n = 2; n <= std::min<int64_t>(16, max_n); ++n) consider(n);
  for (int64_t k = 1; k * x.slots <= kSplitWgsMany; ++k) {
    for (const int pairing : {kMirrored, kSingle, kShort}) {
      const int64_t n = k * x.slots / (workgroups_of_rows((int64_t)x.chunk_len * (x.h_q / x.h_kv), pairing) * (int64_t)x.h_kv);
      if (n > 16 && n <= max_n) consider(n);
    }
  }
  std::lock_guard<std::mutex> lock(g_plan_mutex);
  g_plan_keys[g_plan_next] = key;
  g_plan_values[g_plan_next] = best;
  g_plan_next = (g_plan_next + 1) % kPlanCache;
  if (g_plan_count < kPlanCache) ++g_plan_count;
  return best;
}

mocap_status make_plan(int64_t prefix_len, int32_t chunk_len, int32_t h_q, int32_t h_kv,
                       int32_t head_dim, int32_t num_splits, Plan* plan, size_t ws_cap = SIZE_MAX) {
  const int64_t group = h_q / h_kv;
  // The bound on a chunk's size: 2^24 pairs of 128-row units, counted per
  // block of up to two query heads.
  const int64_t hu = group % 2 == 0 ? 2 : 1;
  plan->units = (h_q / hu) * ((((chunk_len * hu + kUnitRows - 1) / kUnitRows) + 1) / 2);
  if (plan->units > (int64_t)1 << 24) return MOCAP_ERR_UNSUPPORTED;
  plan->row_groups = (int)((chunk_len * group + kUnitRows - 1) / kUnitRows);
  plan->pairs = (plan->row_groups + 1) / 2;
  plan->base_wgs = h_kv * plan->pairs;
  plan->prefix_tiles = (prefix_len + kTileKeys - 1) / kTileKeys;
  int cus = 0;
  if (num_splits == 0 && plan->prefix_tiles > 0) {
    const mocap_status st = device_cu_count(&cus);
    if (st != MOCAP_OK) return st;
  }
  const LaunchShape x{prefix_len, chunk_len, h_q, h_kv, head_dim, plan->row_groups, cus};
  plan->n_ranges = choose_ranges(x, plan->base_wgs, plan->prefix_tiles, num_splits, ws_cap);
  plan->own_range = num_splits > 1;
  plan->ws_bytes = workspace_for(plan->n_ranges, chunk_len, h_q, head_dim);
  return MOCAP_OK;
}

mocap_status check_store(const mocap_kv_store* kv) {
  if (kv == nullptr) return MOCAP_ERR_INVALID_ARG;
  if (kv->num_blocks <= 0 || kv->block_size <= 0 || kv->h_kv <= 0 || kv->head_dim <= 0)
    return MOCAP_ERR_INVALID_ARG;
  if (!supported_head_dim(kv->head_dim)) return MOCAP_ERR_UNSUPPORTED;
  if (kv->block_size % kTileKeys != 0) return MOCAP_ERR_UNSUPPORTED;
  return MOCAP_OK;
}

mocap_status check_positions(const mocap_kv_store* kv, int32_t n_table, int64_t start, int32_t len) {
  if (start < 0 || len < 0 || n_table < 0) return MOCAP_ERR_INVALID_ARG;
  // Kernels index positions with 32-bit integers.
  if (start + (int64_t)len > kMaxPositions) return MOCAP_ERR_INVALID_ARG;
  const int64_t end = start + len;
  const int64_t blocks_needed = (end + kv->block_size - 1) / kv->block_size;
  if (blocks_needed > n_table) return MOCAP_ERR_INVALID_ARG;
  return MOCAP_OK;
}

// Checks shared by the attention entry points (first store, sizes, pointers).
mocap_status check_attn_args(const mocap_kv_store* kv, const int32_t* block_table, int32_t n_table, const void* q,
                             int64_t prefix_len, int32_t chunk_len, int32_t h_q, int32_t h_kv, int32_t head_dim,
                             float scale, const void* o, const float* lse, int32_t num_splits) {
  mocap_status st = check_store(kv);
  if (st != MOCAP_OK) return st;
  if (h_q <= 0 || h_kv <= 0 || h_q % h_kv != 0 || h_kv != kv->h_kv || head_dim != kv->head_dim)
    return MOCAP_ERR_INVALID_ARG;
  if (!(scale > 0.f) || !std::isfinite(scale)) return MOCAP_ERR_INVALID_ARG;
  if (num_splits < 0) return MOCAP_ERR_INVALID_ARG;
  st = check_positions(kv, n_table, prefix_len, chunk_len);
  if (st != MOCAP_OK) return st;
  if (chunk_len == 0) return MOCAP_OK;
  if (!kv->k_pool || !kv->v_pool || !block_table || !q || !o || !lse) return MOCAP_ERR_INVALID_ARG;
  if (!aligned16(kv->k_pool) || !aligned16(kv->v_pool) || !aligned16(block_table) || !aligned16(q) ||
      !aligned16(o) || !aligned16(lse))
    return MOCAP_ERR_INVALID_ARG;
  return MOCAP_OK;
}

// A second store's key range: whole 64-key tiles inside the prefix.
bool valid_remote_range(int64_t begin, int64_t end, int64_t prefix_len) {
  return begin >= 0 && begin <= end && end <= prefix_len && begin % kTileKeys == 0 && end % kTileKeys == 0;
}

// Pairing of row groups for a launch (best_pairing_us), cached per shape.
struct PairKey {
  int64_t prefix_len;
  int32_t chunk_len, h_q, h_kv, head_dim, n_ranges, slots, mode;
  bool own_range;
  bool operator==(const PairKey& o) const {
    return prefix_len == o.prefix_len && chunk_len == o.chunk_len && h_q == o.h_q && h_kv == o.h_kv &&
           head_dim == o.head_dim && n_ranges == o.n_ranges && slots == o.slots && mode == o.mode && own_range == o.own_range;
  }
};
PairKey g_pair_keys[kPlanCache];
int g_pair_values[kPlanCache];
int g_pair_count = 0, g_pair_next = 0;

int choose_pairing(const Plan& plan, int64_t prefix_len, int32_t chunk_len, int32_t h_q, int32_t h_kv,
                    int32_t head_dim, int cus) {
  const PairKey key{prefix_len, chunk_len, h_q, h_kv, head_dim, plan.n_ranges, cus, pairing_mode(),
                    plan.own_range};
  {
    std::lock_guard<std::mutex> lock(g_plan_mutex);
    for (int i = 0; i < g_pair_count; ++i)
      if (g_pair_keys[i] == key) return g_pair_values[i];
  }
  int pairing = kMirrored;
  best_pairing_us(LaunchShape{prefix_len, chunk_len, h_q, h_kv, head_dim, plan.row_groups, std::max(cus, 1)},
                  plan.n_ranges, plan.own_range, &pairing);
  std::lock_guard<std::mutex> lock(g_plan_mutex);
  g_pair_keys[g_pair_next] = key;
  g_pair_values[g_pair_next] = pairing;
  g_pair_next = (g_pair_next + 1) % kPlanCache;
  if (g_pair_count < kPlanCache) ++g_pair_count;
  return pairing;
}

// The launches of one chunk's attention: the attention kernel and, when the
// plan is split, the merge.
struct Prepared {
  mocap::AttnLaunch attn;
  mocap::MergeLaunch merge;
  int32_t head_dim;
};

// Makes the launch descriptions; nothing is enqueued.  Arguments have been
// validated; remote_kv is used only for the plan's second-store ranges.
mocap_status prepare_attention(const mocap_kv_store* kv, const int32_t* block_table, const mocap_kv_store* remote_kv,
                               const int32_t* remote_table, const Plan& plan, const void* q, int64_t prefix_len,
                               int32_t chunk_len, int32_t h_q, int32_t h_kv, int32_t head_dim, float scale,
                               void* o, float* lse, void* workspace, size_t workspace_bytes, Prepared* out) {
  if (plan.units * plan.n_ranges > 0x7fffffff) return MOCAP_ERR_UNSUPPORTED;
  if (plan.n_ranges > 1) {
    if (workspace == nullptr || !aligned16(workspace) || workspace_bytes < plan.ws_bytes)
      return MOCAP_ERR_WORKSPACE;
  }

  out->head_dim = head_dim;
  mocap::AttnLaunch& p = out->attn;
  p.q = static_cast<const uint16_t*>(q);
  p.k_pool = static_cast<const uint16_t*>(kv->k_pool);
  p.v_pool = static_cast<const uint16_t*>(kv->v_pool);
  p.table = block_table;
  p.k_pool_r = remote_kv ? static_cast<const uint16_t*>(remote_kv->k_pool) : nullptr;
  p.v_pool_r = remote_kv ? static_cast<const uint16_t*>(remote_kv->v_pool) : nullptr;
  p.table_r = remote_kv ? remote_table : nullptr;
  p.o = static_cast<uint16_t*>(o);
  p.lse = lse;
  p.prefix_len = (int32_t)prefix_len;
  p.chunk_len = chunk_len;
  p.h_q = h_q;
  p.h_kv = h_kv;
  p.group = h_q / h_kv;
  block_divider((uint32_t)p.group, &p.group_magic, &p.group_shift);
  p.row_groups = plan.row_groups;
  {
    int cus = 0;
    const mocap_status st = device_cu_count(&cus);
    if (st != MOCAP_OK) return st;
    p.pairing = choose_pairing(plan, prefix_len, chunk_len, h_q, h_kv, head_dim, cus);
  }
  p.pairs = workgroups_of_rows((int64_t)chunk_len * p.group, p.pairing);
  const int64_t total = (int64_t)p.pairs * h_kv * plan.n_ranges;
  if (total > 0x7fffffff) return MOCAP_ERR_UNSUPPORTED;
  p.block_size = kv->block_size;
  block_divider((uint32_t)kv->block_size, &p.block_magic, &p.block_shift);
  p.n_ranges = plan.n_ranges;
  p.span_parts = plan.own_range ? plan.n_ranges - 1 : plan.n_ranges;
  p.span_end = (int32_t)(plan.own_range ? prefix_len : prefix_len + chunk_len);
  p.span_tiles = (int32_t)(((int64_t)p.span_end + kTileKeys - 1) / kTileKeys);
  p.remote_begin = (int32_t)plan.remote_begin;
  p.remote_end = (int32_t)plan.remote_end;
  p.total_wgs = (int)total;
  p.scale_log2 = (float)((double)scale * 1.4426950408889634);
  p.ws_o = nullptr;
  p.ws_lse = nullptr;
  if (plan.n_ranges > 1) {
    const size_t rows = (size_t)plan.n_ranges * (size_t)h_q * (size_t)chunk_len;
    p.ws_o = static_cast<float*>(workspace);
    p.ws_lse = reinterpret_cast<float*>(static_cast<char*>(workspace) +
                                        round_up(rows * (size_t)head_dim * sizeof(float), 256));
  }
  mocap::MergeLaunch& m = out->merge;
  m.ws_o = p.ws_o;
  m.ws_lse = p.ws_lse;
  m.o = p.o;
  m.lse = lse;
  m.chunk_len = chunk_len;
  m.h_q = h_q;
  m.n_ranges = plan.n_ranges;
  return MOCAP_OK;
}

mocap_status launch_attention(const Prepared& x, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  const hipError_t launched = x.attn.pairing == kShort ? mocap::launch_chunk_attn_short(x.attn, x.head_dim, s)
                                                       : mocap::launch_chunk_attn(x.attn, x.head_dim, s);
  if (launched != hipSuccess) return MOCAP_ERR_HIP;
  if (x.merge.n_ranges > 1 && mocap::launch_lse_merge(x.merge, x.head_dim, s) != hipSuccess) return MOCAP_ERR_HIP;
  return MOCAP_OK;
}

mocap_status enqueue_attention(const mocap_kv_store* kv, const int32_t* block_table, const mocap_kv_store* remote_kv,
                               const int32_t* remote_table, const Plan& plan, const void* q, int64_t prefix_len,
                               int32_t chunk_len, int32_t h_q, int32_t h_kv, int32_t head_dim, float scale,
                               void* o, float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  Prepared x;
  const mocap_status st = prepare_attention(kv, block_table, remote_kv, remote_table, plan, q, prefix_len, chunk_len,
                                            h_q, h_kv, head_dim, scale, o, lse, workspace, workspace_bytes, &x);
  return st == MOCAP_OK ? launch_attention(x, stream) : st;
}

// Checks of mocap_kv_append.
mocap_status check_append_args(const mocap_kv_store* kv, const int32_t* block_table, int32_t n_table,
                               int64_t start_pos, int32_t chunk_len, const void* k_chunk, const void* v_chunk) {
  mocap_status st = check_store(kv);
  if (st != MOCAP_OK) return st;
  st = check_positions(kv, n_table, start_pos, chunk_len);
  if (st != MOCAP_OK) return st;
  if (chunk_len == 0) return MOCAP_OK;
  if (!kv->k_pool || !kv->v_pool || !block_table || !k_chunk || !v_chunk) return MOCAP_ERR_INVALID_ARG;
  if (!aligned16(kv->k_pool) || !aligned16(kv->v_pool) || !aligned16(block_table) ||
      !aligned16(k_chunk) || !aligned16(v_chunk))
    return MOCAP_ERR_INVALID_ARG;
  return MOCAP_OK;
}

mocap_status launch_append(const mocap_kv_store* kv, const int32_t* block_table, int64_t start_pos, int32_t chunk_len,
                           const void* k_chunk, const void* v_chunk, void* stream) {
  mocap::AppendLaunch p;
  p.k_chunk = static_cast<const uint16_t*>(k_chunk);
  p.v_chunk = static_cast<const uint16_t*>(v_chunk);
  p.k_pool = static_cast<uint16_t*>(kv->k_pool);
  p.v_pool = static_cast<uint16_t*>(kv->v_pool);
  p.table = block_table;
  p.start_pos = start_pos;
  p.chunk_len = chunk_len;
  p.h_kv = kv->h_kv;
  p.block_size = kv->block_size;
  if (mocap::launch_kv_append(p, kv->head_dim, static_cast<hipStream_t>(stream)) != hipSuccess)
    return MOCAP_ERR_HIP;
  return MOCAP_OK;
}

// Host-side check of the block-table entries that positions [first, end) use:
// each in [0, num_blocks), no two logical blocks on one physical block.
mocap_status check_table_entries(const int32_t* table, int32_t n_table, int64_t first, int64_t end,
                                 int32_t block_size, int32_t num_blocks, int32_t* bad_out) {
  if (bad_out) *bad_out = -1;
  if (first < 0 || end < first || block_size <= 0 || num_blocks <= 0 || n_table < 0) return MOCAP_ERR_INVALID_ARG;
  if (end == first) return MOCAP_OK;
  const int64_t b0 = first / block_size, b1 = (end + block_size - 1) / block_size;
  if (b1 > n_table || table == nullptr) return MOCAP_ERR_INVALID_ARG;
  std::vector<std::pair<int32_t, int64_t>> used;
  used.reserve((size_t)(b1 - b0));
  for (int64_t b = b0; b < b1; ++b) {
    if (table[b] < 0 || table[b] >= num_blocks) {
      if (bad_out) *bad_out = (int32_t)b;
      return MOCAP_ERR_INVALID_ARG;
    }
    used.emplace_back(table[b], b);
  }
  std::sort(used.begin(), used.end());
  for (size_t i = 1; i < used.size(); ++i) {
    if (used[i].first == used[i - 1].first) {
      if (bad_out) *bad_out = (int32_t)used[i].second;
      return MOCAP_ERR_INVALID_ARG;
    }
  }
  return MOCAP_OK;
}

// In a build with MOCAP_DEBUG_TABLES, every call copies the table entries it
// will use to the host (a synchronous copy) and checks them before anything
// is enqueued; a bad entry returns MOCAP_ERR_INVALID_ARG.
#ifdef MOCAP_DEBUG_TABLES
mocap_status debug_check_table(const int32_t* dev_table, int64_t first, int64_t end, const mocap_kv_store* kv) {
  if (end <= first) return MOCAP_OK;
  const int64_t b0 = first / kv->block_size, b1 = (end + kv->block_size - 1) / kv->block_size;
  std::vector<int32_t> host((size_t)b1, 0);
  if (hipMemcpy(host.data() + b0, dev_table + b0, (size_t)(b1 - b0) * sizeof(int32_t), hipMemcpyDeviceToHost) !=
      hipSuccess)
    return MOCAP_ERR_HIP;
  return check_table_entries(host.data(), (int32_t)b1, first, end, kv->block_size, kv->num_blocks, nullptr);
}
#define MOCAP_DEBUG_CHECK(table, first, end, kv)                              \
  do {                                                                        \
    const mocap_status debug_st_ = debug_check_table((table), (first), (end), (kv)); \
    if (debug_st_ != MOCAP_OK) return debug_st_;                              \
  } while (0)
#else
#define MOCAP_DEBUG_CHECK(table, first, end, kv) \
  do {                                           \
  } while (0)
#endif

// ---- Scratch of the allocation-free entry point ----
// Split partials of mocap_chunk_attn_noalloc live in this array: every device
// the library runs on holds its own copy until the process ends.  Host code
// never uses the array's name as an address: the device address comes from
// hipGetSymbolAddress, once per device, with that device current.
constexpr size_t kScratchBytes = MOCAP_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
std::atomic<void*> g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mutex;

mocap_status device_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MOCAP_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return MOCAP_ERR_UNSUPPORTED;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    ptr = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (ptr == nullptr) {
      if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return MOCAP_ERR_HIP;
      g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
  }
  *out = ptr;
  return MOCAP_OK;
}

}  // namespace

extern "C" {

const char* mocap_status_string(mocap_status status) {
  switch (status) {
    case MOCAP_OK: return "MOCAP_OK";
    case MOCAP_ERR_INVALID_ARG: return "MOCAP_ERR_INVALID_ARG";
    case MOCAP_ERR_UNSUPPORTED: return "MOCAP_ERR_UNSUPPORTED";
    case MOCAP_ERR_WORKSPACE: return "MOCAP_ERR_WORKSPACE";
    case MOCAP_ERR_HIP: return "MOCAP_ERR_HIP";
  }
  return "MOCAP_ERR_UNKNOWN";
}

mocap_status mocap_kv_append(const mocap_kv_store* kv, const int32_t* block_table, int32_t n_table,
                             int64_t start_pos, int32_t chunk_len, const void* k_chunk,
                             const void* v_chunk, void* stream) {
  const mocap_status st = check_append_args(kv, block_table, n_table, start_pos, chunk_len, k_chunk, v_chunk);
  if (st != MOCAP_OK || chunk_len == 0) return st;
  MOCAP_DEBUG_CHECK(block_table, start_pos, start_pos + chunk_len, kv);
  return launch_append(kv, block_table, start_pos, chunk_len, k_chunk, v_chunk, stream);
}

mocap_status mocap_chunk_attn_workspace_size(int64_t prefix_len, int32_t chunk_len, int32_t h_q,
                                             int32_t h_kv, int32_t head_dim, int32_t num_splits,
                                             int32_t* splits_out, size_t* bytes_out) {
  if (bytes_out == nullptr) return MOCAP_ERR_INVALID_ARG;
  if (prefix_len < 0 || chunk_len < 0 || h_q <= 0 || h_kv <= 0 || h_q % h_kv != 0 || num_splits < 0)
    return MOCAP_ERR_INVALID_ARG;
  if (prefix_len + (int64_t)chunk_len > kMaxPositions) return MOCAP_ERR_INVALID_ARG;
  if (!supported_head_dim(head_dim)) return MOCAP_ERR_UNSUPPORTED;
  if (chunk_len == 0) {
    if (splits_out) *splits_out = 1;
    *bytes_out = 0;
    return MOCAP_OK;
  }
  Plan plan;
  const mocap_status st = make_plan(prefix_len, chunk_len, h_q, h_kv, head_dim, num_splits, &plan);
  if (st != MOCAP_OK) return st;
  if (splits_out) *splits_out = plan.n_ranges;
  *bytes_out = plan.ws_bytes;
  return MOCAP_OK;
}

mocap_status mocap_chunk_attn(const mocap_kv_store* kv, const int32_t* block_table, int32_t n_table,
                              const void* q, int64_t prefix_len, int32_t chunk_len, int32_t h_q,
                              int32_t h_kv, int32_t head_dim, float scale, void* o, float* lse,
                              void* workspace, size_t workspace_bytes, int32_t num_splits,
                              void* stream) {
  mocap_status st = check_attn_args(kv, block_table, n_table, q, prefix_len, chunk_len, h_q, h_kv, head_dim,
                                    scale, o, lse, num_splits);
  if (st != MOCAP_OK || chunk_len == 0) return st;
  MOCAP_DEBUG_CHECK(block_table, 0, prefix_len + chunk_len, kv);
  Plan plan;
  st = make_plan(prefix_len, chunk_len, h_q, h_kv, head_dim, num_splits, &plan);
  if (st != MOCAP_OK) return st;
  return enqueue_attention(kv, block_table, nullptr, nullptr, plan, q, prefix_len, chunk_len, h_q, h_kv,
                           head_dim, scale, o, lse, workspace, workspace_bytes, stream);
}

mocap_status mocap_chunk_prefill(const mocap_kv_store* kv, const int32_t* block_table, int32_t n_table,
                                 const int32_t* lengths, int32_t num_chunks, const void* q, const void* k,
                                 const void* v, int32_t h_q, int32_t h_kv, int32_t head_dim, float scale, void* o,
                                 float* lse, void* workspace, size_t workspace_bytes, int32_t num_splits,
                                 void* stream) {
  mocap_status st = check_store(kv);
  if (st != MOCAP_OK) return st;
  if (num_chunks < 0 || (num_chunks > 0 && lengths == nullptr) || h_q <= 0) return MOCAP_ERR_INVALID_ARG;
  const int64_t q_row = (int64_t)h_q * head_dim, kv_row = (int64_t)kv->h_kv * kv->head_dim;
  // Null stays null, for the checks to refuse.
  auto row = [](const void* base, int64_t elems) -> const void* {
    return base ? static_cast<const uint16_t*>(base) + elems : nullptr;
  };
  int32_t used = 0;  // chunks that are not empty
  for (int32_t c = 0; c < num_chunks; ++c) used += lengths[c] != 0;
  std::unique_ptr<Prepared[]> prepared(new (std::nothrow) Prepared[used]);
  if (!prepared) return MOCAP_ERR_UNSUPPORTED;
  // Every chunk is checked and prepared before the first one is enqueued.
  int64_t prefix = 0, lse_at = 0;
  Prepared* x = prepared.get();
  for (int32_t c = 0; c < num_chunks; ++c) {
    const int32_t n = lengths[c];
    const void* q_c = row(q, prefix * q_row);
    void* o_c = const_cast<void*>(row(o, prefix * q_row));
    float* lse_c = lse ? lse + lse_at : nullptr;
    st = check_append_args(kv, block_table, n_table, prefix, n, row(k, prefix * kv_row), row(v, prefix * kv_row));
    if (st != MOCAP_OK) return st;
    st = check_attn_args(kv, block_table, n_table, q_c, prefix, n, h_q, h_kv, head_dim, scale, o_c, lse_c, num_splits);
    if (st != MOCAP_OK) return st;
    if (n == 0) continue;
    Plan plan;
    st = make_plan(prefix, n, h_q, h_kv, head_dim, num_splits, &plan);
    if (st != MOCAP_OK) return st;
    st = prepare_attention(kv, block_table, nullptr, nullptr, plan, q_c, prefix, n, h_q, h_kv, head_dim, scale, o_c,
                           lse_c, workspace, workspace_bytes, x++);
    if (st != MOCAP_OK) return st;
    prefix += n;
    lse_at += ((int64_t)h_q * n + 3) / 4 * 4;
  }
  MOCAP_DEBUG_CHECK(block_table, 0, prefix, kv);
  for (const Prepared* y = prepared.get(); y < x; ++y) {
    const int64_t at = y->attn.prefix_len * kv_row;
    st = launch_append(kv, block_table, y->attn.prefix_len, y->attn.chunk_len, row(k, at), row(v, at), stream);
    if (st != MOCAP_OK) return st;
    st = launch_attention(*y, stream);
    if (st != MOCAP_OK) return st;
  }
  return MOCAP_OK;
}

mocap_status mocap_check_block_table(const int32_t* block_table, int32_t n_table, int64_t first_pos,
                                     int64_t end_pos, int32_t block_size, int32_t num_blocks,
                                     int32_t* bad_index_out) {
  return check_table_entries(block_table, n_table, first_pos, end_pos, block_size, num_blocks, bad_index_out);
}

mocap_status mocap_chunk_attn_noalloc(const mocap_kv_store* kv, const int32_t* block_table, int32_t n_table,
                                      const void* q, int64_t prefix_len, int32_t chunk_len, int32_t h_q,
                                      int32_t h_kv, int32_t head_dim, float scale, void* o, float* lse,
                                      int32_t num_splits, void* stream) {
  mocap_status st = check_attn_args(kv, block_table, n_table, q, prefix_len, chunk_len, h_q, h_kv, head_dim,
                                    scale, o, lse, num_splits);
  if (st != MOCAP_OK || chunk_len == 0) return st;
  MOCAP_DEBUG_CHECK(block_table, 0, prefix_len + chunk_len, kv);
  Plan plan;
  st = make_plan(prefix_len, chunk_len, h_q, h_kv, head_dim, num_splits, &plan, kScratchBytes);
  if (st != MOCAP_OK) return st;
  if (plan.ws_bytes > kScratchBytes) return MOCAP_ERR_WORKSPACE;  // a forced split that does not fit
  void* ws = nullptr;
  if (plan.n_ranges > 1) {
    st = device_scratch(&ws);
    if (st != MOCAP_OK) return st;
  }
  return enqueue_attention(kv, block_table, nullptr, nullptr, plan, q, prefix_len, chunk_len, h_q, h_kv, head_dim,
                           scale, o, lse, ws, kScratchBytes, stream);
}

mocap_status mocap_chunk_attn_two_store_workspace_size(int64_t prefix_len, int32_t chunk_len, int32_t h_q,
                                                       int32_t h_kv, int32_t head_dim, int64_t remote_begin,
                                                       int64_t remote_end, int32_t num_splits,
                                                       int32_t* splits_out, size_t* bytes_out) {
  if (bytes_out == nullptr) return MOCAP_ERR_INVALID_ARG;
  if (prefix_len < 0 || chunk_len < 0 || h_q <= 0 || h_kv <= 0 || h_q % h_kv != 0 || num_splits < 0)
    return MOCAP_ERR_INVALID_ARG;
  if (prefix_len + (int64_t)chunk_len > kMaxPositions) return MOCAP_ERR_INVALID_ARG;
  if (!supported_head_dim(head_dim)) return MOCAP_ERR_UNSUPPORTED;
  if (!valid_remote_range(remote_begin, remote_end, prefix_len)) return MOCAP_ERR_INVALID_ARG;
  if (chunk_len == 0) {
    if (splits_out) *splits_out = 1;
    *bytes_out = 0;
    return MOCAP_OK;
  }
  Plan plan;
  const mocap_status st = make_plan(prefix_len, chunk_len, h_q, h_kv, head_dim, num_splits, &plan);
  if (st != MOCAP_OK) return st;
  if (splits_out) *splits_out = plan.n_ranges;
  *bytes_out = plan.ws_bytes;
  return MOCAP_OK;
}

mocap_status mocap_chunk_attn_two_store(const mocap_kv_store* kv, const int32_t* block_table, int32_t n_table,
                                        const mocap_kv_store* remote_kv, const int32_t* remote_table,
                                        int32_t n_remote_table, int64_t remote_begin, int64_t remote_end,
                                        const void* q, int64_t prefix_len, int32_t chunk_len, int32_t h_q,
                                        int32_t h_kv, int32_t head_dim, float scale, void* o, float* lse,
                                        void* workspace, size_t workspace_bytes, int32_t num_splits,
                                        void* stream) {
  mocap_status st = check_attn_args(kv, block_table, n_table, q, prefix_len, chunk_len, h_q, h_kv, head_dim,
                                    scale, o, lse, num_splits);
  if (st != MOCAP_OK) return st;
  if (!valid_remote_range(remote_begin, remote_end, prefix_len)) return MOCAP_ERR_INVALID_ARG;
  if (remote_begin == remote_end) {
    if (chunk_len == 0) return MOCAP_OK;
    MOCAP_DEBUG_CHECK(block_table, 0, prefix_len + chunk_len, kv);
    Plan plan;
    st = make_plan(prefix_len, chunk_len, h_q, h_kv, head_dim, num_splits, &plan);
    if (st != MOCAP_OK) return st;
    return enqueue_attention(kv, block_table, nullptr, nullptr, plan, q, prefix_len, chunk_len, h_q, h_kv,
                             head_dim, scale, o, lse, workspace, workspace_bytes, stream);
  }
  st = check_store(remote_kv);
  if (st != MOCAP_OK) return st;
  if (remote_kv->h_kv != kv->h_kv || remote_kv->head_dim != kv->head_dim ||
      remote_kv->block_size != kv->block_size)
    return MOCAP_ERR_INVALID_ARG;
  st = check_positions(remote_kv, n_remote_table, 0, (int32_t)remote_end);
  if (st != MOCAP_OK) return st;
  if (chunk_len == 0) return MOCAP_OK;
  if (!remote_kv->k_pool || !remote_kv->v_pool || !remote_table || !aligned16(remote_kv->k_pool) ||
      !aligned16(remote_kv->v_pool) || !aligned16(remote_table))
    return MOCAP_ERR_INVALID_ARG;
  MOCAP_DEBUG_CHECK(block_table, 0, remote_begin, kv);
  MOCAP_DEBUG_CHECK(block_table, remote_end, prefix_len + chunk_len, kv);
  MOCAP_DEBUG_CHECK(remote_table, remote_begin, remote_end, remote_kv);
  Plan plan;
  st = make_plan(prefix_len, chunk_len, h_q, h_kv, head_dim, num_splits, &plan);
  if (st != MOCAP_OK) return st;
  plan.remote_begin = remote_begin / kTileKeys;
  plan.remote_end = remote_end / kTileKeys;
  return enqueue_attention(kv, block_table, remote_kv, remote_table, plan, q, prefix_len, chunk_len, h_q, h_kv,
                           head_dim, scale, o, lse, workspace, workspace_bytes, stream);
}

}  // extern "C"
