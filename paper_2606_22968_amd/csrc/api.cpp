// Host side of libmocap_attn's device calls: argument validation, split
// planning and kernel dispatch.  Every check runs before anything is
// enqueued.  The host-only chunk planners live in plan.cpp.
#include "mocap_attn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <bitset>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
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
  int pairing;       // -1: not chosen with the ranges
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

// The model above.  A caller whose prefix moves plans on every call, so this
// has to stay short of the launch it plans.  Almost all workgroups of a launch
// cost the same: costs are made as they are handed out, the compute units'
// finishing times stay in a sorted ring (a new one goes in near its end), and
// bounds made without any of that leave few candidates to walk through.
// Planning a new shape, up to 512 tokens behind up to 10^6 keys: 12 us on
// average, 63 at the 99th percentile; with an array of all costs and a heap for
// every candidate 72 and 450.  Up to 8192 tokens: 18 us against 92.
class LaunchModel {
 public:
  LaunchModel(const LaunchShape& x, bool own_range)
      : x_(x), group_(x.h_q / x.h_kv), rows_((int64_t)x.chunk_len * group_), own_(own_range),
        all_tiles_((x.prefix_len + x.chunk_len + kTileKeys - 1) / kTileKeys),
        span_(own_range ? (x.prefix_len + kTileKeys - 1) / kTileKeys : all_tiles_),
        xcd_slots_(std::min(std::max(1, x.slots / kXcds), kRing)),
        tile_us_(x.head_dim == 128 ? kTileUs128 : kTileUs64), group_us_(x.head_dim == 128 ? kGroupUs128 : kGroupUs64),
        step_us_(x.head_dim == 128 ? kStepUs128 : kStepUs64) {
    for (int pairing : {kMirrored, kAdjacent, kSingle, kShort}) lay_out(pairing);
  }

  // The best placement of row groups in workgroups (mirrored: q with R-1-q,
  // every workgroup about equally long, the units sharing the tiles only the
  // longer one sees; adjacent: 2q with 2q+1, both units on their own rows nearly
  // throughout, workgroups of different lengths evened out when there are many
  // per compute unit; single: both units on one row group's tiles, half of each
  // tile's keys, which pays where even then compute units stay free; short: the
  // other kernel).  In this order, another one only when the model expects it to
  // win clearly over the best so far.  Returns its time, or infinity if no
  // placement stays under `limit`; with us_out null the time is not made.
  int best(int n_ranges, double limit, int forced, double* us_out) const {
    if (forced >= 0) {
      if (us_out) *us_out = bound(forced, n_ranges) < limit ? estimate(forced, n_ranges, limit) : INFINITY;
      return forced;
    }
    // With up to two row groups the two ways to pair them are the same, with
    // one so is single.
    const int64_t groups = layout_[kMirrored].units;
    const bool open[4] = {true, groups > 2, groups > 1 && few_enough(kSingle, n_ranges),
                          few_enough(kShort, n_ranges)};
    constexpr double bar[4] = {1.0, 0.98, 0.98, 0.95};
    double lo[4], hi[4];  // the time lies between
    double least = INFINITY;
    for (int p = kMirrored; p <= kShort; ++p) {
      lo[p] = hi[p] = INFINITY;
      if (!open[p]) continue;
      lo[p] = bound(p, n_ranges);
      if (limit < INFINITY) {
        const double us = lo[p] < limit ? estimate(p, n_ranges, limit) : INFINITY;
        lo[p] = us < INFINITY ? us : std::max(lo[p], limit);
        hi[p] = us;
      } else {
        hi[p] = upper_bound(p, n_ranges);
      }
      least = std::min(least, lo[p]);
    }
    if (least >= limit) {
      if (us_out) *us_out = INFINITY;
      return kMirrored;
    }
    auto settle = [&](int p) { lo[p] = hi[p] = estimate(p, n_ranges, INFINITY); };
    // The last one that wins over every one before it; then one by one.
    int best = kMirrored;
    double before = lo[kMirrored];
    for (int p = kAdjacent; p <= kShort; ++p) {
      if (open[p] && hi[p] < bar[p] * before) best = p;
      before = std::min(before, lo[p]);
    }
    for (int p = best + 1; p <= kShort; ++p) {
      if (!open[p]) continue;
      while (hi[p] >= bar[p] * lo[best] && lo[p] < bar[p] * hi[best] && (lo[best] < hi[best] || lo[p] < hi[p]))
        settle(lo[best] < hi[best] ? best : p);
      if (hi[p] < bar[p] * lo[best]) best = p;
    }
    if (us_out) {
      if (lo[best] < hi[best]) settle(best);
      *us_out = hi[best];
    }
    return best;
  }

  // A lower bound of the time of any placement.
  double least(int n_ranges) const {
    double us = INFINITY;
    for (int p : {kMirrored, kAdjacent, kSingle, kShort})
      if (few_enough(p, n_ranges)) us = std::min(us, bound(p, n_ranges));
    return us;
  }

 private:
  static constexpr int kRing = 256;  // compute units of an XCD, at most

  struct Layout {
    int64_t units;  // row groups, or 32-row slots (short)
    int64_t wgs;    // workgroups of one KV head and range
    bool lone;      // the last of them has one row group where the others have two
    double work;    // tiles of one KV head's workgroups over the whole span, in units of kTileUs
  };

  bool few_enough(int pairing, int64_t n_ranges) const {
    const int64_t rounds = pairing == kSingle ? kSingleRounds : pairing == kShort ? kShortRounds : INT64_MAX / x_.slots;
    return layout_[pairing].wgs * x_.h_kv * n_ranges <= rounds * x_.slots;
  }

  // The end of the tiles that row group (or slot) u sees.
  int64_t unit_end(int64_t u, int unit_rows) const {
    const int64_t tokens = std::min<int64_t>(x_.chunk_len, ((u + 1) * unit_rows + group_ - 1) / group_);
    return (x_.prefix_len + tokens + kTileKeys - 1) / kTileKeys;
  }
  static int unit_rows(int pairing) { return pairing == kShort ? kAttnWaveRows : kUnitRows; }

  // The row groups of workgroup q (the lower one -1: none): q and R-1-q, R-2-2q
  // and R-1-2q, or R-1-q alone.
  void groups_of(int pairing, int64_t q, int64_t* top, int64_t* other) const {
    const int64_t last = layout_[pairing].units - 1;
    *top = pairing == kAdjacent ? last - 2 * q : last - q;
    *other = pairing >= kSingle ? -1 : pairing == kAdjacent ? *top - 1 : q < *top ? q : -1;
  }

  // Cost of a workgroup whose row groups see a and b of a range's tiles (b = 0: alone).
  double cost_of(int pairing, int64_t a, int64_t b) const {
    if (pairing == kShort) return (double)((2 * a + kAttnWaves - 1) / kAttnWaves) * step_us_ + kShortGroupUs;
    return ((double)b + (double)(a - b) * kLoneTile) * tile_us_ + group_us_;
  }

  void lay_out(int pairing) {
    Layout& l = layout_[pairing];
    l.units = (rows_ + unit_rows(pairing) - 1) / unit_rows(pairing);
    l.wgs = workgroups_of_rows(rows_, pairing);
    l.lone = pairing < kSingle && l.units % 2 != 0;
    // Sum over the span: its ranges cover each row group's tiles once (the tile
    // of the prefix's end twice if the chunk's keys are a range of their own).
    const int64_t twice = own_ ? span_ - x_.prefix_len / kTileKeys : 0;
    l.work = 0.0;
    if (!few_enough(pairing, 1)) return;  // is never looked at
    for (int64_t q = 0; q < l.wgs; ++q) {
      int64_t top, other;
      groups_of(pairing, q, &top, &other);
      const double a = (double)(unit_end(top, unit_rows(pairing)) + twice);
      const double b = other >= 0 ? (double)(unit_end(other, unit_rows(pairing)) + twice) : 0.0;
      l.work += pairing == kShort ? a : b + (a - b) * kLoneTile;
    }
  }

  double stream_us(int pairing) const {
    return kStreamWeight * (4.0 * (x_.prefix_len + x_.chunk_len) * x_.h_kv * x_.head_dim /
                            (pairing == kShort ? kShortBytesPerUs : kTileBytesPerUs));
  }
  double fixed_us(int n_ranges) const {
    if (n_ranges <= 1) return kLaunchUs;
    const double partial = (double)n_ranges * x_.chunk_len * x_.h_q * (x_.head_dim + 1) * 4.0;
    return kLaunchUs + 2.0 * partial / kMergeBytesPerUs + kLaunchUs;
  }
  static double total_us(double fixed, double makespan, double stream) {
    return fixed + std::sqrt(makespan * makespan + stream * stream);
  }

  // At least the mean load of a compute unit; and the ranges that every row
  // sees in full cost the same up to one tile, so some compute unit gets a
  // whole number of those.
  double bound(int pairing, int n_ranges) const {
    const Layout& l = layout_[pairing];
    const double per_tile = pairing == kShort ? 2.0 / kAttnWaves * step_us_ : tile_us_;
    const double per_wg = pairing == kShort ? kShortGroupUs : group_us_;
    double load = (l.work * per_tile + (double)(l.wgs * n_ranges) * per_wg) * x_.h_kv / (xcd_slots_ * kXcds);
    const int64_t parts = own_ ? n_ranges - 1 : n_ranges;
    if (parts > 0 && l.wgs > 0) {
      const int64_t seen = x_.prefix_len / kTileKeys + 1;  // tiles that every row sees
      const int64_t inner = own_ ? parts : std::min<int64_t>(parts, ((seen + 1) * parts - 1) / span_);
      // Those with a pair of row groups, and all of them at the cost of the lone one.
      const int64_t tiles = span_ / parts;
      auto least_of = [&](int64_t wgs, bool pair) {
        const int64_t jobs = inner * wgs * x_.h_kv;
        const int64_t rounds = ((jobs + kXcds - 1) / kXcds + xcd_slots_ - 1) / xcd_slots_;
        const int64_t t = tiles + (rounds == 1 && span_ % parts > parts - inner ? 1 : 0);
        load = std::max(load, (double)rounds * cost_of(pairing, t, pair ? t : 0));
      };
      if (pairing < kSingle && l.wgs > (l.lone ? 1 : 0)) least_of(l.wgs - (l.lone ? 1 : 0), true);
      if (pairing >= kSingle || l.lone) least_of(l.wgs, false);
    }
    // Rounding of the sums aside.
    return total_us(fixed_us(n_ranges), load, stream_us(pairing)) * (1.0 - 1e-9);
  }

  // At most: the longest workgroup behind the mean of as many of them.
  double upper_bound(int pairing, int n_ranges) const {
    const Layout& l = layout_[pairing];
    const int64_t parts = own_ ? n_ranges - 1 : n_ranges;
    int64_t tiles = parts > 0 ? (span_ + parts - 1) / parts : 0;
    if (own_) tiles = std::max(tiles, all_tiles_ - x_.prefix_len / kTileKeys);
    const double longest = cost_of(pairing, tiles, pairing < kSingle && l.units > 1 ? tiles : 0);
    const int64_t jobs = (l.wgs * n_ranges * x_.h_kv + kXcds - 1) / kXcds;
    const double rounds = jobs <= xcd_slots_ ? 1.0 : (double)jobs / xcd_slots_ + 1.0;
    return total_us(fixed_us(n_ranges), rounds * longest, stream_us(pairing)) * (1.0 + 1e-9);
  }

  // Infinity if it is certain to reach `limit`.
  double estimate(int pairing, int n_ranges, double limit) const {
    const double fixed = fixed_us(n_ranges), stream = stream_us(pairing);
    double longest = INFINITY;  // makespan
    if (limit < INFINITY) {
      const double rest = limit - fixed;
      if (rest <= stream) return INFINITY;
      longest = std::sqrt(rest * rest - stream * stream) * (1.0 + 1e-9);
    }
    const double makespan = simulate(pairing, n_ranges, longest);
    return makespan < INFINITY ? total_us(fixed, makespan, stream) : INFINITY;
  }

  // The workgroups in the order in which the hardware hands them out; infinity
  // if one ends after `longest`.
  double simulate(int pairing, int n_ranges, double longest) const {
    const Layout& l = layout_[pairing];
    const int64_t size = l.wgs * n_ranges;  // workgroups of one KV head
    const int64_t total = size * x_.h_kv;
    const int64_t parts = own_ ? n_ranges - 1 : n_ranges;
    const int64_t seen = x_.prefix_len / kTileKeys + 1;
    const int rows = unit_rows(pairing);
    std::pair<int64_t, int64_t> done[kXcds];  // (first workgroup of its KV head, count) of the XCDs so far
    double makespan = 0.0;
    double ring[kRing];
    int64_t next = 0;
    for (int xcd = 0; xcd < kXcds; ++xcd) {
      const int64_t count = total / kXcds + (xcd < total % kXcds ? 1 : 0);
      done[xcd] = {next % size, count};
      next += count;
      if (std::find(done, done + xcd, done[xcd]) != done + xcd) continue;  // runs the same workgroups
      int head = 0, busy = 0;  // ring[head ..] holds `busy` times in ascending order
      auto hand_out = [&](double t) {
        if (busy == xcd_slots_) {
          t += ring[head];
          head = (head + 1) & (kRing - 1);
        } else {
          ++busy;
        }
        int at = (head + busy - 1) & (kRing - 1);
        for (int i = busy - 1; i > 0; --i) {
          const int before = (at + kRing - 1) & (kRing - 1);
          if (ring[before] <= t) break;
          ring[at] = ring[before];
          at = before;
        }
        ring[at] = t;
      };
      int64_t r = done[xcd].first / l.wgs, q = done[xcd].first % l.wgs;
      for (int64_t left = count; left > 0;) {
        const int64_t t0 = r < parts ? span_ * r / parts : x_.prefix_len / kTileKeys;
        const int64_t t1 = r < parts ? span_ * (r + 1) / parts : all_tiles_;
        const int64_t stop = q + std::min(l.wgs - q, left);
        left -= stop - q;
        const bool inner = t1 <= seen;
        const double full = cost_of(pairing, t1 - t0, pairing < kSingle ? t1 - t0 : 0);
        for (; q < stop; ++q) {
          if (inner && !(l.lone && q == l.wgs - 1)) {
            hand_out(full);
            continue;
          }
          int64_t top, other;
          groups_of(pairing, q, &top, &other);
          const int64_t a = std::max<int64_t>(0, std::min(t1, unit_end(top, rows)) - t0);
          const int64_t b = other >= 0 ? std::max<int64_t>(0, std::min(t1, unit_end(other, rows)) - t0) : 0;
          hand_out(cost_of(pairing, a, b));
        }
        if (busy > 0 && ring[(head + busy - 1) & (kRing - 1)] > longest) return INFINITY;
        q = 0;
        r = r + 1 == n_ranges ? 0 : r + 1;
      }
      if (busy > 0) makespan = std::max(makespan, ring[(head + busy - 1) & (kRing - 1)]);
    }
    return makespan;
  }

  const LaunchShape& x_;
  const int64_t group_, rows_;
  const bool own_;
  const int64_t all_tiles_, span_;
  const int xcd_slots_;
  const double tile_us_, group_us_, step_us_;
  Layout layout_[4];
};

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
std::pair<int, int> g_plan_values[kPlanCache];  // ranges, pairing
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
int choose_ranges(const LaunchShape& x, int base_wgs, int64_t prefix_tiles, int requested, size_t ws_cap,
                  int* pairing_out) {
  *pairing_out = -1;
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
      if (g_plan_keys[i] == key) {
        *pairing_out = g_plan_values[i].second;
        return g_plan_values[i].first;
      }
  }
  const LaunchModel model(x, false);
  const int mode = pairing_mode();
  int best = 1;
  double best_us;
  int pairing = model.best(1, INFINITY, mode, &best_us);
  best_us *= 0.98;  // a split must pay for itself clearly
  std::bitset<kSplitWgsMany + 1> tried;  // counts above 8 are at most kSplitWgsMany
  auto consider = [&](int64_t n) {
    if (tried[(size_t)n] || workspace_for((int)n, x.chunk_len, x.h_q, x.head_dim) > ws_cap) return;
    tried[(size_t)n] = true;
    double us;
    const int with = model.best((int)n, best_us, mode, &us);
    if (us < best_us || (us == best_us && best > 1 && n < best)) {
      best_us = us;
      best = (int)n;
      pairing = with;
    }
  };
  const int64_t all_tiles = (x.prefix_len + x.chunk_len + kTileKeys - 1) / kTileKeys;
  const int64_t max_n = std::min(all_tiles / kMinRangeTiles,
                                 std::max(std::min(kFewRanges, kSplitWgsFew / base_wgs), kSplitWgsMany / base_wgs));
  auto each_count = [&](auto&& visit) {
    for (int64_t n = 2; n <= std::min<int64_t>(16, max_n); ++n) visit(n);
    for (int64_t k = 1; max_n > 16 && k * x.slots <= kSplitWgsMany; ++k) {
      for (const int p : {kMirrored, kSingle, kShort}) {
        const int64_t n = k * x.slots / (workgroups_of_rows((int64_t)x.chunk_len * (x.h_q / x.h_kv), p) * (int64_t)x.h_kv);
        if (n > 16 && n <= max_n) visit(n);
      }
    }
  };
  // The most promising count first: what it takes rules most others out.
  int64_t first = 0;
  double first_us = INFINITY;
  each_count([&](int64_t n) {
    const double us = model.least((int)n);
    if (us < first_us) {
      first_us = us;
      first = n;
    }
  });
  if (first > 0) consider(first);
  each_count(consider);
  std::lock_guard<std::mutex> lock(g_plan_mutex);
  g_plan_keys[g_plan_next] = key;
  g_plan_values[g_plan_next] = {best, pairing};
  g_plan_next = (g_plan_next + 1) % kPlanCache;
  if (g_plan_count < kPlanCache) ++g_plan_count;
  *pairing_out = pairing;
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
  plan->n_ranges = choose_ranges(x, plan->base_wgs, plan->prefix_tiles, num_splits, ws_cap, &plan->pairing);
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

// Pairing of row groups for a launch whose ranges were not chosen here, cached per shape.
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
  const LaunchShape x{prefix_len, chunk_len, h_q, h_kv, head_dim, plan.row_groups, std::max(cus, 1)};
  const int pairing = LaunchModel(x, plan.own_range).best(plan.n_ranges, INFINITY, pairing_mode(), nullptr);
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
  p.pairing = plan.pairing;
  if (p.pairing < 0) {
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
