// C-ABI entry points: argument validation, work planning and launches.
//
// Every check runs on the host before the first HIP call, so a bad call
// returns an error with nothing enqueued.  Planning is host arithmetic only:
// sequences are ordered longest first, the (row tile, key split) units of
// each sequence are numbered longest first, and the kv-head index varies
// fastest over workgroup ids -- workgroups are dispatched round-robin over the
// 8 XCDs, so with 8 (or a multiple/divisor of 8) kv-heads every workgroup of
// one kv-head runs on the same XCD and its K/V stream is shared in that L2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <numeric>
#include <unordered_set>
#include <vector>

#include "kvt.h"
#include "kvt_internal.h"

namespace {

thread_local int g_last_hip_error = 0;

kvt_status device_error(hipError_t e) {
  g_last_hip_error = (int)e;
  return KVT_ERR_DEVICE;
}

int elem_bytes(int32_t dtype) { return dtype == KVT_DTYPE_BF16 ? 2 : 4; }

// Number of compute units of the current device, queried once per device
// (concurrent first calls may both query; they store the same value).
int device_cus() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return 256; }
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
      (void)hipGetLastError();
      n = 256;
    }
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// The kernels move 16-byte pieces of every token row, page and workspace.
bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

kvt_status check_pool(const kvt_pool* pool) {
  if (pool == nullptr || pool->k == nullptr || pool->v == nullptr) return KVT_ERR_INVALID_ARG;
  if (!aligned16(pool->k) || !aligned16(pool->v)) return KVT_ERR_INVALID_ARG;
  if (pool->num_blocks < 1 || pool->num_kv_heads < 1) return KVT_ERR_INVALID_ARG;
  if (pool->head_dim != 64 && pool->head_dim != 128) return KVT_ERR_UNSUPPORTED;
  if (pool->dtype != KVT_DTYPE_BF16 && pool->dtype != KVT_DTYPE_F32) return KVT_ERR_UNSUPPORTED;
  return KVT_OK;
}

// Validates lengths and table width; fills the total token count.
kvt_status check_seqs(const kvt_seqs* seqs, int64_t* total_tokens) {
  if (seqs == nullptr || seqs->num_seqs < 1) return KVT_ERR_INVALID_ARG;
  if (seqs->prefix_len == nullptr || seqs->suffix_len == nullptr || seqs->block_table == nullptr)
    return KVT_ERR_INVALID_ARG;
  if (seqs->max_blocks < 1) return KVT_ERR_INVALID_ARG;
  int64_t T = 0;
  for (int b = 0; b < seqs->num_seqs; ++b) {
    const int64_t P = seqs->prefix_len[b], S = seqs->suffix_len[b];
    if (P < 0 || S < 1) return KVT_ERR_INVALID_ARG;
    const int64_t L = P + S;
    if (L > INT32_MAX / 2) return KVT_ERR_INVALID_ARG;
    if ((L + kvt::kBlock - 1) / kvt::kBlock > seqs->max_blocks) return KVT_ERR_INVALID_ARG;
    T += S;
  }
  if (T > INT32_MAX / 2) return KVT_ERR_INVALID_ARG;
  *total_tokens = T;
  return KVT_OK;
}

// Query heads: a positive multiple of the kv-heads, and T * num_q_heads
// packed query rows must fit the kernels' 32-bit row indices.
bool heads_ok(const kvt_pool* pool, int32_t num_q_heads, int64_t T) {
  if (num_q_heads < 1 || num_q_heads % pool->num_kv_heads != 0) return false;
  return T * num_q_heads <= INT32_MAX;
}

// Checked mode: every used block id is inside the pool.
kvt_status check_table_ids(const kvt_pool* pool, const kvt_seqs* seqs) {
  if (seqs->block_table_host == nullptr) return KVT_OK;
  for (int b = 0; b < seqs->num_seqs; ++b) {
    const int64_t L = (int64_t)seqs->prefix_len[b] + seqs->suffix_len[b];
    const int64_t nblk = (L + kvt::kBlock - 1) / kvt::kBlock;
    const int32_t* row = seqs->block_table_host + (int64_t)b * seqs->max_blocks;
    for (int64_t i = 0; i < nblk; ++i)
      if (row[i] < 0 || (int64_t)row[i] >= pool->num_blocks) return KVT_ERR_OUT_OF_RANGE;
  }
  return KVT_OK;
}

bool overlaps(const void* a, size_t an, const void* b, size_t bn) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + bn && y < x + an;
}

// Workspace of nsplit partial results per packed row: the unnormalised
// outputs in fp32 (256-byte aligned block), then (m, l) in fp32.
size_t part_o_bytes(const kvt_pool* pool, int nsplit, int64_t rows) {
  return (((size_t)nsplit * rows * pool->head_dim * sizeof(float) + 255) / 256) * 256;
}
size_t part_bytes(const kvt_pool* pool, int nsplit, int64_t rows) {
  return part_o_bytes(pool, nsplit, rows) + (size_t)nsplit * rows * 2 * sizeof(float);
}

struct ExtendPlan {
  int nsplit = 1;
  int nsplit_base = 1;      // splits to fall back to when the workspace offered is too small for nsplit
  int nsplit_shared = 0;    // cascade only: key splits of the shared part
  bool use_shared = true;   // cascade only: false = run the plain extend plan
  double heaviest = 0.0;    // extend only: weight of the heaviest row tile when lighter ones take fewer splits, else 0
  std::vector<int> order;   // sequences, longest key range first
  size_t ws_bytes = 0;      // workspace needed for nsplit > 1
};

int row_tiles(int32_t suffix, int group) {
  const int64_t rows = (int64_t)suffix * group;
  return (int)((rows + kvt::kExtTileRows - 1) / kvt::kExtTileRows);
}

// Cost of the combine launch that merges split partials, in us.
constexpr double kMergeLaunchUs = 4.0;
// Fixed cost of one workgroup, in key tiles: its prologue (kernel arguments,
// block-table entries and the first tile's gather, about 3.3 us) and its
// epilogue.
constexpr double kUnitTiles = 2.0;

// CUs by the time they become free, as runs of equal times in ascending
// order, so that equal units on equally free CUs are placed in one step.  (A
// heap of the CUs is filled and popped unit by unit: it was most of the time
// of a cascade's plan.)
class FreeTimes {
 public:
  FreeTimes(double early, int64_t n_early, double late, int64_t n_late) {
    if (n_early > 0) runs_.push_back({early, n_early});
    if (n_late > 0) runs_.push_back({late, n_late});
  }
  // Puts `jobs` units of length len, one after the other, each on the CU that
  // is free first; returns the latest finish.
  double run(int64_t jobs, double len) {
    double last = 0;
    while (jobs > 0) {
      Run& first = runs_[head_];
      const int64_t n = std::min(jobs, first.count);
      const double t = first.time + len;
      jobs -= n;
      if ((first.count -= n) == 0) ++head_;
      auto at = std::lower_bound(runs_.begin() + head_, runs_.end(), t, [](const Run& r, double x) { return r.time < x; });
      if (at != runs_.end() && at->time == t) at->count += n;
      else runs_.insert(at, Run{t, n});
      last = t;   // the earliest free CU never gets earlier
    }
    return last;
  }

 private:
  struct Run {
    double time;
    int64_t count;
  };
  std::vector<Run> runs_;
  size_t head_ = 0;
};

// Finish time, in key tiles, of one extend launch: list scheduling of its
// units in launch order onto the CUs (each unit to the CU that frees first,
// as workgroups are dispatched): shared_jobs units of len_s tiles first
// (a cascade's shared part; none for a plain extend), then each sequence's
// units (jobs_p[b] row tiles of ceil(kt_p[b] / ns_p) tiles, ns_p splits
// each, of which one in `share` falls to the CUs modelled); every unit also
// pays kUnitTiles.  Callers model one kv-head's units on its share of the
// CUs (the units of the kv-heads alternate) or one XCD's (workgroups go to
// the XCDs in turn).
double list_finish(int64_t shared_jobs, double len_s, const std::vector<int64_t>& jobs_p,
                   const std::vector<int64_t>& kt_p, int ns_p, int cus, int share = 1) {
  const int64_t rounds = shared_jobs / cus, rest = shared_jobs % cus;
  const double early = (double)rounds * (len_s + kUnitTiles), late = (double)(rounds + 1) * (len_s + kUnitTiles);
  FreeTimes free_at(early, cus - rest, late, rest);
  double span = rest > 0 ? late : early;
  for (size_t b = 0; b < jobs_p.size(); ++b) {
    const double len = std::ceil((double)kt_p[b] / ns_p) + kUnitTiles;
    span = std::max(span, free_at.run((jobs_p[b] * ns_p + share - 1) / share, len));
  }
  return span;
}

// Sequences in launch order, longest key range first (stable).
std::vector<int> longest_first(const kvt_seqs* seqs) {
  std::vector<int> order(seqs->num_seqs);
  std::iota(order.begin(), order.end(), 0);
  if (order.size() > 1)
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
      return (int64_t)seqs->prefix_len[x] + seqs->suffix_len[x] > (int64_t)seqs->prefix_len[y] + seqs->suffix_len[y];
    });
  return order;
}

// Split long key ranges only when the row tiles alone cannot fill the chip.
ExtendPlan make_plan(const kvt_pool* pool, const kvt_seqs* seqs, int32_t num_q_heads, int64_t T, int cus) {
  ExtendPlan p;
  const int B = seqs->num_seqs;
  const int G = num_q_heads / pool->num_kv_heads;
  p.order = longest_first(seqs);
  int64_t units = 0;
  int64_t min_keys = INT64_MAX, min_len = INT64_MAX, max_len = 0;
  for (int b = 0; b < B; ++b) {
    units += (int64_t)row_tiles(seqs->suffix_len[b], G) * pool->num_kv_heads;
    min_keys = std::min<int64_t>(min_keys, (int64_t)seqs->prefix_len[b] + 1);
    const int64_t len = (int64_t)seqs->prefix_len[b] + seqs->suffix_len[b];
    min_len = std::min(min_len, len);
    max_len = std::max(max_len, len);
  }
  // Split the key range when whole rounds of workgroups over the CUs leave
  // many CUs idle: with ns splits a unit's work shrinks to 1/ns and the call
  // takes about ceil(units*ns / cus) / ns unit-times.  Take the smallest ns
  // with the best estimate if it beats no split by at least 10 %; each split
  // keeps at least 16 key tiles (1024 keys) of the shortest sequence.
  const int64_t by_keys = std::max<int64_t>(1, min_keys / (16 * kvt::kExtKeysPerTile));
  const int ns_max = (int)std::min<int64_t>(by_keys, kvt::kMaxSplits);
  auto rounds = [&](int s) { return (double)((units * s + cus - 1) / cus) / s; };
  int ns = 1;
  for (int s = 2; s <= ns_max; ++s)
    if (rounds(s) < rounds(ns) - 1e-9) ns = s;
  if (rounds(ns) > 0.9 * rounds(1)) ns = 1;
  // Ragged batches: the rule above counts units as equal and keeps 1024 keys
  // of the shortest sequence per split, so one short sequence stops the long
  // ones from splitting.  When the longest key range is more than twice the
  // shortest and the row tiles fit a few rounds of the CUs, list-schedule
  // the launch for 1, 2, 4, 8 and 16 splits (one XCD's eighth of the units
  // on its CUs, each unit's length from its sequence's key tiles) and take
  // the best finish plus partial cost if it beats the rule's choice by more
  // than a fifth.
  constexpr int kXcds = 8;
  const int xcd_cus = std::max(1, cus / kXcds);
  if (max_len > 2 * min_len && units <= 4 * (int64_t)cus) {
    const int64_t rows = T * num_q_heads;
    std::vector<int64_t> jobs(B), kt(B);
    for (int i = 0; i < B; ++i) {
      const int b = p.order[i];
      jobs[i] = (int64_t)row_tiles(seqs->suffix_len[b], G) * pool->num_kv_heads;
      kt[i] = ((int64_t)seqs->prefix_len[b] + seqs->suffix_len[b] + kvt::kExtKeysPerTile - 1) / kvt::kExtKeysPerTile;
    }
    auto cost = [&](int s) {
      double t = list_finish(0, 0.0, jobs, kt, s, xcd_cus, kXcds);
      if (s > 1) t += (2.0 * (double)part_bytes(pool, s, rows) / 5.0e6 + kMergeLaunchUs) / 1.8;
      return t;
    };
    const double rule_cost = cost(ns);
    int best = ns;
    double best_cost = rule_cost;
    for (int s = 1; s <= kvt::kMaxSplits; s *= 2) {
      const double c = cost(s);
      if (c < best_cost - 1e-9) best = s, best_cost = c;
    }
    if (best_cost < 0.8 * rule_cost) ns = best;
  }
  p.nsplit = p.nsplit_base = ns;
  if (ns > 1) p.ws_bytes = part_bytes(pool, ns, T * num_q_heads);
  return p;
}

// Weight of one key tile of the last row tile of a sequence against a full
// one's, by its waves that hold rows: up to four have a SIMD each to
// themselves (1.05 us per key tile with eight workgroups running, 1.42 to 1.63
// with all CUs busy on keys of their own), from five on they share SIMDs
// (1.41 to 1.50, 1.93 to 2.40).
constexpr double kTileWeight[3] = {0.65, 0.95, 1.0};
int last_tile_class(int32_t suffix, int group) {
  const int64_t rows = (int64_t)suffix * group % kvt::kExtTileRows;
  if (rows == 0) return 2;
  return rows <= 4 * kvt::kExtRowsPerWave ? 0 : 1;
}

// Key splits of a last row tile of one class: fewer than the full row tiles
// take when it is lighter, so that every unit takes about as long.
int last_splits(int nsplit, double heaviest, int tile_class) {
  if (heaviest == 0.0 || kTileWeight[tile_class] == heaviest) return nsplit;
  return std::max(1, (int)std::lround(nsplit * kTileWeight[tile_class] / heaviest));
}

// The split plan of an extend call is make_plan's, unless the call has at most
// one row tile per CU and like contexts (the longest at most twice the
// shortest): then refine_plan looks further.  make_plan counts every row tile
// as full and keeps 1024 keys per split, which leaves most of the chip idle for
// a short message over a few thousand keys; here the row tiles of one kv-head,
// each with its weight, are laid over that head's share of the CUs for a range
// of split counts (up to kMaxPartials, down to one key tile per split), every
// unit charged its key tiles, kUnitTiles, and every round of units in full, and
// the merge charged 4.5 us and its partials at 4.5 TB/s.  The best is taken if
// it beats make_plan's count by more than 5 %, and an unsplit one also by 6 key
// tiles (the second launch and the workspace cost the host about 5 us, the
// device a launch gap).  Plans whose partials would no longer fit the no-alloc
// entry point's static scratch where make_plan's do are left alone: one plan
// serves both entry points, and what the no-alloc one took it takes.  Per pass, make_plan's count and this one: 37 new tokens over 2000
// keys, 32/8 heads, 51.1 and 29.3 us; 64 over 131072, 24/2 heads, 196 and
// 113 us; 67 over 30011, 32/8 heads, 61.1 and 56.8 us; 20 over 700 keys (left
// alone) 24 and 29 us.
void refine_plan(ExtendPlan* p, const kvt_pool* pool, const kvt_seqs* seqs, int32_t num_q_heads, int64_t T, int cus) {
  const int B = seqs->num_seqs, G = num_q_heads / pool->num_kv_heads;
  const int64_t rows = T * num_q_heads;
  const int longest = p->order.front(), shortest = p->order.back();
  const int64_t max_len = (int64_t)seqs->prefix_len[longest] + seqs->suffix_len[longest];
  const int64_t min_len = (int64_t)seqs->prefix_len[shortest] + seqs->suffix_len[shortest];
  const int head_cus = cus / pool->num_kv_heads;
  if (max_len > 2 * min_len || B > head_cus) return;
  int64_t tiles = 0;   // row tiles of one kv-head: full ones, and last ones by class
  int last[3] = {0, 0, 0};
  double heaviest = 0.0;
  for (int b = 0; b < B; ++b) {
    const int t = row_tiles(seqs->suffix_len[b], G), c = last_tile_class(seqs->suffix_len[b], G);
    tiles += t;
    ++last[c];
    heaviest = std::max(heaviest, t > 1 ? 1.0 : kTileWeight[c]);
  }
  if (tiles > head_cus) return;
  const int full = (int)tiles - B;
  const int kt = (int)((max_len + kvt::kExtKeysPerTile - 1) / kvt::kExtKeysPerTile);
  auto cost = [&](int ns, bool weighted) {
    int units = full * ns;   // at most 64 per CU
    for (int c = 0; c < 3; ++c)
      if (last[c] > 0) units += last[c] * (weighted ? last_splits(ns, heaviest, c) : ns);
    const double unit = heaviest * (double)((kt + ns - 1) / ns) + kUnitTiles;
    const double merge = ns > 1 ? (4.5 + (double)part_bytes(pool, ns, rows) / 4.5e6) / 1.8 : 0.0;
    return (double)((units + head_cus - 1) / head_cus) * unit + merge;
  };
  const double base = cost(p->nsplit, false);
  int best = 0;
  double best_cost = 0.95 * base - (p->nsplit == 1 ? 6.0 : 0.0);
  double per_split = (double)full;   // units per split count
  for (int b = 0; b < B; ++b) per_split += kTileWeight[last_tile_class(seqs->suffix_len[b], G)] / heaviest;
  auto consider = [&](int ns) {
    if (ns < 1 || ns > kvt::kMaxPartials || ns > kt) return;
    const double c = cost(ns, true);
    if (c < best_cost - 1e-9) best = ns, best_cost = c;
  };
  for (int ns = 1; ns <= kvt::kMaxPartials; ns *= 2) consider(ns);
  for (int r = 1; r <= 3; ++r)   // the counts that fill whole rounds (or just do, where rounding adds a unit)
    for (int ns = (int)(r * head_cus / per_split), k = 0; k < 2; ++k) consider(ns - k);
  if (best == 0) return;
  const size_t bytes = best > 1 ? part_bytes(pool, best, rows) : 0;
  if (bytes > (size_t)KVT_NOALLOC_SCRATCH_BYTES && p->ws_bytes <= (size_t)KVT_NOALLOC_SCRATCH_BYTES) return;
  p->nsplit = best;
  p->heaviest = heaviest;
  p->ws_bytes = bytes;
}

ExtendPlan extend_plan(const kvt_pool* pool, const kvt_seqs* seqs, int32_t num_q_heads, int64_t T) {
  const int cus = device_cus();
  ExtendPlan p = make_plan(pool, seqs, num_q_heads, T, cus);
  refine_plan(&p, pool, seqs, num_q_heads, T, cus);
  return p;
}

// Keys of a decoding batch (each sequence's new one included).
int64_t total_keys(const kvt_seqs* seqs) {
  int64_t total = seqs->num_seqs;
  for (int b = 0; b < seqs->num_seqs; ++b) total += seqs->prefix_len[b];
  return total;
}

// Workgroups of a decode launch that share a CU: 0 for as many as fit (two with
// heads of 128; four with heads of 64, three in fp32), else fewer.  Where one
// has a CU to itself, units run longest first, each at the CU's full rate, and
// short ones fill the CUs that become free.  Where several share it, the first
// units share the bandwidth as well, and when the shorter ones have ended, the
// longest are too few to use it.  `reach` is how much of a step the longest
// unit takes at half a CU; `mean` is the mean unit's keys.
//   * Unlike contexts: one per CU from reach 1.05 on (from 1.5 on in split
//     plans of 3.5 and more units per CU; with bf16 heads of 64 in split plans
//     and below 3000 keys a unit), if units are long enough to hide a
//     workgroup's start and end without a neighbour (below that from 2.4 on).
//     Per step, two per CU and one, 96/8 heads of 128: 64 contexts of
//     1000..8192 keys (reach 2.6) 147.9, 129.8 us; 90 of 2000..32768 (2.4)
//     615.7, 537.2; 128 of 1000..8192 (1.3) 258.8, 256.3; 100 of 1000..8192 in
//     two splits (0.8) 219.1, 229.7; 32 of 2048..32768 in four (1.4) 242.0,
//     244.5; 48 in three (1.6) 279.0, 272.7; 28 of 13000..39800 in three (1.15,
//     672 units) 434.1, 413.7; 48 of 500..4096 in two (1.8, 850 keys a unit)
//     53.2, 57.5.  Otherwise at most two: 32/8 heads of 64, four and two: 160
//     of 1000..8192 158.2, 153.5; 128 of 500..4096 69.8, 65.0; but 256 of
//     100..600 31.8, 38.6.
//   * Like contexts fill whole rounds, so what the last round (of two per CU)
//     leaves decides: 90 of 4000..8000 keys (208 units in it) 341.9, 319.4 us;
//     48 in two splits (256) 188.3, 180.8; but 72 (64 units) 263.4, 273.0; 100
//     (288) 373.5, 383.2; 64 (none) 237.8, 230.6.  With four per CU, a last
//     round that is nearly full, or lengths that differ, in the first: heads of
//     64, four and two: 100 of 2000..4000 keys (800 units) 102.4, 94.5; 112 of
//     4000..8000 (896) 212.1, 206.3; 72 of 4000..8000 (reach 1.2) 145.4, 136.3;
//     but 72 of 4096 (0.9) 105.1, 119.6; 200 of 4000..8000 (576) 375.7, 388.0.
int decode_per_cu(const kvt_pool* pool, const kvt_seqs* seqs, const ExtendPlan& plan) {
  const int64_t cus = device_cus(), units = (int64_t)seqs->num_seqs * plan.nsplit * pool->num_kv_heads;
  if (units <= cus) return 0;
  const int64_t max_keys = (int64_t)seqs->prefix_len[plan.order.front()] + 1;
  const int64_t min_keys = (int64_t)seqs->prefix_len[plan.order.back()] + 1;
  const double longest = (double)max_keys / plan.nsplit;
  const double mean = (double)total_keys(seqs) / ((double)seqs->num_seqs * plan.nsplit);
  const double reach = 2.0 * longest / (mean * (double)units / (double)cus);
  if (max_keys > 2 * min_keys) {
    if (mean < 1500) return mean >= 800 && reach >= 2.4 ? 1 : 0;
    const bool late = pool->head_dim == 64 && pool->dtype == KVT_DTYPE_BF16
                          ? plan.nsplit > 1 || mean < 3000
                          : plan.nsplit > 1 && 2 * units >= 7 * cus;
    return reach >= (late ? 1.5 : 1.05) ? 1 : 2;
  }
  if (mean < 1500) return 0;
  if (pool->head_dim == 64) {
    if (pool->dtype != KVT_DTYPE_BF16) return 0;
    return units % (4 * cus) >= 3 * cus || (units < 4 * cus && reach >= 1.1) ? 2 : 0;
  }
  const int64_t rest = units % (2 * cus);
  return (rest == 0 && reach >= 1.35) || (2 * rest >= cus && rest <= cus && reach >= 0.9) ? 1 : 0;
}

// Decode: one unit per (sequence, key split) and kv-head.  Splits are added
// while the workgroups cannot cover the CUs twice over (two share a CU), at
// most kMaxSplits, keeping at least 1024 keys of the shortest sequence per
// split (each of the 4 waves then streams at least 8 tiles of 32 keys).
// Beside that base count:
//   * a small batch of like contexts (the longest at most twice the shortest)
//     would leave CUs idle; its splits fill the CUs once, down to 128 keys
//     per split (one tile per wave), at most kMaxPartials.  One context,
//     kernel + merge: 131072 keys of 8 kv-heads 98.3 + 4.3 us at 16 splits,
//     81.8 + 4.9 at 32 (256 workgroups), 88.2 + 7.5 at 64; 2048 keys 17.1 + 2.4
//     at 2, 9.6 + 2.6 at 8, 8.2 + 3.0 at 16.  Where the base count is 1 that
//     adds the merge, so the splits have to take 400 keys (heads of 64: 500)
//     from the longest workgroup: 8 kv-heads, unsplit and split, 16 contexts of
//     600 keys (2 splits) 12.6, 13.8 us, of 1300 20.8, 19.9; 8 of 600 (4) 12.2,
//     12.1, of 1000 16.0, 12.8; with heads of 64 16 of 600 8.3, 9.6, of 1300
//     12.9, 12.2.  In fp32 half the CUs already reach the bandwidth: two splits
//     of 16 contexts of 1700 keys 36.2, 39.5, heads of 64 19.5, 22.5;
//   * from one unit per CU on, if a unit of the longest context takes longer
//     than a CU's mean share of the keys, the longest contexts decide when the
//     step ends; with two rounds of workgroups (four per CU in all) and at
//     least 4096 keys of the longest per split, the rest fills in beside them.
//     So it does if like contexts leave a last round (of two per CU) nearly
//     empty, and in any batch where only one workgroup fits a CU (fp32 heads
//     of 128: 36 contexts of 2091..16734 keys 569 us at 2 splits, 550 at 4).
//     Per step of 32 contexts at 2, 3, 4, 6 splits: 2048..32768 keys 287, 260,
//     247, 251 us; 16384..32768 keys (the longest unit 0.7 of a CU's share)
//     497, 514, 490, 503 us; 64 contexts of 8192 keys (0.5) at 1 and 2: 325,
//     342 us; 70 (48 workgroups in the last round) 396, 383; 80 (128) 413, 428.
ExtendPlan make_decode_plan(const kvt_pool* pool, const kvt_seqs* seqs, int32_t num_q_heads) {
  ExtendPlan p;
  const int B = seqs->num_seqs;
  p.order.resize(B);
  std::iota(p.order.begin(), p.order.end(), 0);
  std::stable_sort(p.order.begin(), p.order.end(),
                   [&](int x, int y) { return seqs->prefix_len[x] > seqs->prefix_len[y]; });
  const int64_t max_keys = (int64_t)seqs->prefix_len[p.order.front()] + 1;
  const int64_t min_keys = (int64_t)seqs->prefix_len[p.order.back()] + 1;
  const int64_t units = (int64_t)B * pool->num_kv_heads;
  const int64_t cus = device_cus();
  const bool like = max_keys <= 2 * min_keys;
  const int64_t want = (2 * cus + units - 1) / units;
  const int64_t by_keys = std::max<int64_t>(1, min_keys / 1024);
  p.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>({want, by_keys, (int64_t)kvt::kMaxSplits}));
  p.nsplit_base = p.nsplit;
  if (like) {
    const int64_t fill = std::min<int64_t>({cus / units, min_keys / 128, (int64_t)kvt::kMaxPartials});
    const bool pays = max_keys * (fill - 1) >= (pool->head_dim == 64 ? 500 : 400) * fill &&
                      (fill > 2 || pool->dtype == KVT_DTYPE_BF16);
    if (p.nsplit > 1 || pays) p.nsplit = (int)std::max<int64_t>(p.nsplit, fill);
  }
  const int64_t rest = units * p.nsplit % (2 * cus);
  const bool one_fits = pool->dtype == KVT_DTYPE_F32 && pool->head_dim == 128;
  if (units >= cus && (one_fits || max_keys * cus >= total_keys(seqs) * pool->num_kv_heads * p.nsplit ||
                       (like && rest > 0 && 2 * rest < cus))) {
    const int64_t rounds = (4 * cus + units / 2) / units;   // to the nearest
    p.nsplit = (int)std::max<int64_t>(p.nsplit, std::min(rounds, max_keys / 4096));
  }
  if (p.nsplit > 1) p.ws_bytes = part_bytes(pool, p.nsplit, (int64_t)B * num_q_heads);
  return p;
}

// Fits a plan to the workspace a call offers: the plan itself when it fits,
// unsplit when none is offered, and else the base split count, which asks
// for no more than any call with these arguments ever had to offer: where it
// is unsplit, any workspace argument will do.
kvt_status fit_workspace(ExtendPlan* plan, const kvt_pool* pool, int64_t rows, const void* workspace,
                         size_t workspace_bytes) {
  if (plan->nsplit == 1) return KVT_OK;
  if (workspace == nullptr && workspace_bytes == 0) {
    plan->nsplit = 1;   // no scratch offered: run unsplit
    plan->heaviest = 0.0;
    return KVT_OK;
  }
  if (workspace != nullptr && workspace_bytes >= plan->ws_bytes && aligned16(workspace)) return KVT_OK;
  plan->nsplit = plan->nsplit_base;
  plan->heaviest = 0.0;
  if (plan->nsplit == 1) return KVT_OK;
  plan->ws_bytes = part_bytes(pool, plan->nsplit, rows);
  if (workspace == nullptr || workspace_bytes < plan->ws_bytes) return KVT_ERR_WORKSPACE;
  return aligned16(workspace) ? KVT_OK : KVT_ERR_INVALID_ARG;
}

// A shared prefix: a positive multiple of 16 no longer than any sequence's
// prefix; in checked mode every table row must list the same pages for it.
kvt_status check_shared(const kvt_seqs* seqs, int32_t shared_len) {
  if (shared_len < kvt::kBlock || shared_len % kvt::kBlock != 0) return KVT_ERR_INVALID_ARG;
  for (int b = 0; b < seqs->num_seqs; ++b)
    if (seqs->prefix_len[b] < shared_len) return KVT_ERR_INVALID_ARG;
  if (seqs->block_table_host != nullptr) {
    const int32_t* row0 = seqs->block_table_host;
    for (int b = 1; b < seqs->num_seqs; ++b)
      if (std::memcmp(row0, seqs->block_table_host + (int64_t)b * seqs->max_blocks,
                      sizeof(int32_t) * (shared_len / kvt::kBlock)) != 0)
        return KVT_ERR_INVALID_ARG;
  }
  return KVT_OK;
}

// Estimated time of one extend launch in units of one 64-key tile of one
// 256-row workgroup: the larger of the work spread over the CUs and the
// longest unit's share of its key splits, plus the split partials written
// and read back when split.
double launch_estimate(const kvt_seqs* seqs, int group, int kv_heads, int nsplit, int64_t rows, const kvt_pool* pool,
                       int cus) {
  // one tile of one workgroup takes about 1.8 us at full load; the partials
  // move at about 5 TB/s (written once, read once by the combine),
  // and the combine launch itself costs about 4 us
  constexpr double kTileUs = 1.8, kBytesPerUs = 5.0e6;
  double work = 0, longest = 0;
  for (int b = 0; b < seqs->num_seqs; ++b) {
    const int64_t kt = ((int64_t)seqs->prefix_len[b] + seqs->suffix_len[b] + kvt::kExtKeysPerTile - 1) /
                       kvt::kExtKeysPerTile;
    work += (double)((int64_t)row_tiles(seqs->suffix_len[b], group) * kv_heads) * kt;
    longest = std::max(longest, (double)kt);
  }
  double t = std::max(work / cus, longest / nsplit) + kUnitTiles;
  if (nsplit > 1) t += (2.0 * (double)part_bytes(pool, nsplit, rows) / kBytesPerUs + kMergeLaunchUs) / kTileUs;
  return t;
}

// Cascade: the split plans of the shared part (one virtual sequence of all T
// new tokens over the shared keys, all visible) and of the private parts
// (prefix lengths less the shared prefix); the workspace holds one partial
// per split of either part.  The shared pass reads the shared keys once per
// packed row tile of the whole batch instead of once per sequence's row
// tiles, but every row then goes through partials and a merge; when the
// estimate says the plain extend is faster (long suffixes, where row tiles
// pack well anyway), the plan is the plain extend's (use_shared = false).
//
// The choice is made with make_plan's split counts; the route that runs is then
// refined as a short message's plan is (refine_plan; the shared pass unless
// `base`, and if the estimate gains more than 5 %).  Host time of a plan: 4.5
// us for 24 forks on one kv-head, 2.7 for 16 on eight (26.3 and 18.7 with both
// routes refined and every unit through a heap of the CUs, 9.2 and 14.5 with
// that heap before there was anything to refine).
// 3 sequences adding 3..16 tokens over 4096 shared keys, 32/8 heads: 29.6 us per
// pass with make_plan's count, 25.7 with this; 9 adding 5..20, 24/2 heads, 40.0
// and 33.5.  Calls that fill the chip keep their count (16 over 32768 shared).
ExtendPlan cascade_plan(const kvt_pool* pool, const kvt_seqs* seqs, int32_t shared_len, int32_t num_q_heads,
                        int64_t T, int32_t mode = KVT_CASCADE_AUTO, bool base = false) {
  if (mode == KVT_CASCADE_PLAIN) {
    ExtendPlan plain = extend_plan(pool, seqs, num_q_heads, T);
    plain.use_shared = false;
    return plain;
  }
  const int B = seqs->num_seqs, G = num_q_heads / pool->num_kv_heads, H = pool->num_kv_heads;
  const int KT = kvt::kExtKeysPerTile;
  const int cus = device_cus();
  const int64_t rows = T * num_q_heads;
  std::vector<int32_t> priv(B);
  for (int b = 0; b < B; ++b) priv[b] = seqs->prefix_len[b] - shared_len;
  kvt_seqs ps = *seqs;
  ps.prefix_len = priv.data();
  const int32_t shared_prefix = shared_len - 1, all_tokens = (int32_t)T;
  kvt_seqs ss = *seqs;
  ss.num_seqs = 1;
  ss.prefix_len = &shared_prefix;
  ss.suffix_len = &all_tokens;
  ExtendPlan shared_plan = make_plan(pool, &ss, num_q_heads, T, cus);

  int64_t head_jobs = 0;   // private units of one kv-head
  for (int b = 0; b < B; ++b) head_jobs += row_tiles(seqs->suffix_len[b], G);
  const int head_cus = std::max(1, cus / H);
  const bool one_round = head_jobs <= head_cus;
  ExtendPlan p;
  if (one_round) p.order = longest_first(&ps);   // the split count is placed below
  else p = make_plan(pool, &ps, num_q_heads, T, cus);
  std::vector<int64_t> jobs_p(B), kt_p(B);   // launch order, longest first; one kv-head's units
  for (int i = 0; i < B; ++i) {
    const int b = p.order[i];
    jobs_p[i] = row_tiles(seqs->suffix_len[b], G);
    kt_p[i] = ((int64_t)priv[b] + seqs->suffix_len[b] + KT - 1) / KT;
  }
  const int64_t shared_tiles = row_tiles((int32_t)T, G);
  const double kt_shared = (double)((shared_len + KT - 1) / KT);
  auto partial_cost = [&](int parts) {
    return (2.0 * (double)part_bytes(pool, parts, rows) / 5.0e6 + kMergeLaunchUs) / 1.8;
  };
  // Split counts of both parts with ns_s splits of the shared part, and their
  // estimate.  In one launch the private units can fill what the shared part
  // leaves idle: when one kv-head's private units fit one round of its CUs,
  // their split count is the one (trying 1, 2, 4, 8, 16 until the estimate
  // rises) with the earliest list-scheduled finish plus partial cost.
  auto place = [&](int ns_s, int* ns_p) {
    const int64_t head_shared = shared_tiles * ns_s;
    const double len_s = std::ceil(kt_shared / ns_s);
    if (one_round) {
      int best = 1;
      double t = list_finish(head_shared, len_s, jobs_p, kt_p, 1, head_cus) + partial_cost(ns_s + 1);
      for (int ns = 2; ns <= kvt::kMaxSplits; ns *= 2) {
        const double c = list_finish(head_shared, len_s, jobs_p, kt_p, ns, head_cus) + partial_cost(ns_s + ns);
        if (c >= t - 1e-9) break;
        best = ns, t = c;
      }
      *ns_p = best;
      return t;
    }
    // many private units: the work of both parts spread over the CUs, or
    // the longest unit of either
    double work = (double)(head_shared * H) * len_s, longest = len_s;
    for (int i = 0; i < B; ++i) {
      work += (double)(jobs_p[i] * H) * kt_p[i];
      longest = std::max(longest, (double)kt_p[i] / p.nsplit);
    }
    *ns_p = p.nsplit;
    return std::max(work / cus, longest) + kUnitTiles + partial_cost(ns_s + p.nsplit);
  };
  int ns_p = 1;
  const double t_shared = place(shared_plan.nsplit, &ns_p);

  if (mode == KVT_CASCADE_AUTO) {
    // the choice weighs make_plan's split counts, whatever refine_plan makes of them
    ExtendPlan plain = make_plan(pool, seqs, num_q_heads, T, cus);
    if (!(t_shared < launch_estimate(seqs, G, H, plain.nsplit, rows, pool, cus))) {
      refine_plan(&plain, pool, seqs, num_q_heads, T, cus);
      plain.use_shared = false;
      return plain;
    }
  }
  int ns_s = shared_plan.nsplit;
  if (!base) {
    refine_plan(&shared_plan, pool, &ss, num_q_heads, T, cus);
    const int ns = std::min(shared_plan.nsplit, kvt::kMaxPartials - kvt::kMaxSplits);
    // the shared units alone, with one private set, are a lower bound: place
    // nothing when even they gain too little
    const double len = std::ceil(kt_shared / ns);
    const double least = one_round ? (double)((shared_tiles * ns + head_cus - 1) / head_cus) * (len + kUnitTiles)
                                   : len + kUnitTiles;
    int q = 1;
    if (ns != ns_s && least + partial_cost(ns + 1) < 0.95 * t_shared && place(ns, &q) < 0.95 * t_shared)
      ns_s = ns, ns_p = q;
  }
  p.nsplit_shared = ns_s;
  p.nsplit = ns_p;
  p.ws_bytes = part_bytes(pool, ns_s + ns_p, rows);
  return p;
}

bool mode_ok(int32_t mode) {
  return mode == KVT_CASCADE_AUTO || mode == KVT_CASCADE_SHARED_PASS || mode == KVT_CASCADE_PLAIN;
}

// out must not overlap q or a pool; lse must not overlap out.
kvt_status check_outputs(const kvt_pool* pool, const void* q, int32_t num_q_heads, const void* out,
                         const float* lse, int64_t T) {
  if (!aligned16(q) || !aligned16(out) || ((uintptr_t)lse & 3) != 0) return KVT_ERR_INVALID_ARG;
  const size_t es = elem_bytes(pool->dtype);
  const size_t tok_bytes = (size_t)T * num_q_heads * pool->head_dim * es;
  const size_t pool_bytes = (size_t)pool->num_blocks * pool->num_kv_heads * kvt::kBlock * pool->head_dim * es;
  if (overlaps(out, tok_bytes, q, tok_bytes) || overlaps(out, tok_bytes, pool->k, pool_bytes) ||
      overlaps(out, tok_bytes, pool->v, pool_bytes))
    return KVT_ERR_INVALID_ARG;
  if (lse != nullptr && overlaps(lse, (size_t)T * num_q_heads * sizeof(float), out, tok_bytes))
    return KVT_ERR_INVALID_ARG;
  return KVT_OK;
}

// Launch arguments common to extend and decode.
kvt::ExtendArgs base_args(const kvt_pool* pool, const kvt_seqs* seqs, const void* q, int32_t num_q_heads,
                          float scale, void* out, float* lse, int64_t T, const ExtendPlan& plan, void* workspace) {
  kvt::ExtendArgs a;
  std::memset(&a, 0, sizeof(a));
  a.q = q;
  a.k_pool = pool->k;
  a.v_pool = pool->v;
  a.out = out;
  a.lse = lse;
  a.block_table = seqs->block_table;
  a.num_blocks = pool->num_blocks;
  a.max_blocks = seqs->max_blocks;
  a.num_q_heads = num_q_heads;
  a.num_kv_heads = pool->num_kv_heads;
  a.group = num_q_heads / pool->num_kv_heads;
  a.scale_log2 = scale * 1.4426950408889634f;
  a.kbeg = 0;
  a.kend = INT32_MAX;
  a.direct = plan.nsplit == 1 ? 1 : 0;
  a.part_base = 0;
  a.nsplit = plan.nsplit;
  a.total_rows = (int32_t)T;
  a.second = INT32_MAX;   // one group of sequences
  a.kbeg2 = 0;
  a.kend2 = INT32_MAX;
  a.nsplit2 = 1;
  a.part_base2 = 0;
  if (plan.nsplit > 1) {
    a.part_o = reinterpret_cast<float*>(workspace);
    a.part_ml = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) +
                                         part_o_bytes(pool, plan.nsplit, T * num_q_heads));
  }
  return a;
}

// Merge of the per-split partial results into out (and lse).
kvt_status combine(const kvt::ExtendArgs& a, const kvt_pool* pool, void* out, float* lse, int64_t T,
                   int32_t num_q_heads, int nsplit, bool gaps, hipStream_t s) {
  kvt::CombineArgs c;
  c.part_o = a.part_o;
  c.part_ml = a.part_ml;
  c.out = out;
  c.lse = lse;
  c.rows = T * num_q_heads;
  c.nsplit = nsplit;
  c.gaps = gaps ? 1 : 0;
  const hipError_t e = kvt::launch_combine(c, pool->dtype, pool->head_dim, s);
  return e == hipSuccess ? KVT_OK : device_error(e);
}

// The argument checks of kvt_extend_attention (and its no-alloc variant);
// fills the total token count.
kvt_status check_extend(const kvt_pool* pool, const kvt_seqs* seqs, const void* q, int32_t num_q_heads, float scale,
                        const void* out, const float* lse, int64_t* T) {
  kvt_status st = check_pool(pool);
  if (st != KVT_OK) return st;
  if ((st = check_seqs(seqs, T)) != KVT_OK) return st;
  if (q == nullptr || out == nullptr) return KVT_ERR_INVALID_ARG;
  if (!heads_ok(pool, num_q_heads, *T)) return KVT_ERR_INVALID_ARG;
  if (!(scale > 0.f) || !std::isfinite(scale)) return KVT_ERR_INVALID_ARG;
  if ((st = check_table_ids(pool, seqs)) != KVT_OK) return st;
  return check_outputs(pool, q, num_q_heads, out, lse, *T);
}

// Launches of one extend call under `plan` (partials in `workspace` when split).
kvt_status launch_extend_plan(const kvt_pool* pool, const kvt_seqs* seqs, const void* q, int32_t num_q_heads,
                              float scale, void* out, float* lse, int64_t T, const ExtendPlan& plan,
                              void* workspace, void* stream) {
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int G = num_q_heads / pool->num_kv_heads;
  std::vector<int32_t> row_off(seqs->num_seqs + 1, 0);
  for (int b = 0; b < seqs->num_seqs; ++b) row_off[b + 1] = row_off[b] + seqs->suffix_len[b];

  kvt::ExtendArgs a = base_args(pool, seqs, q, num_q_heads, scale, out, lse, T, plan, workspace);
  for (size_t c0 = 0; c0 < plan.order.size(); c0 += kvt::kSeqsPerLaunch) {
    const int n = (int)std::min<size_t>(kvt::kSeqsPerLaunch, plan.order.size() - c0);
    a.nseq = n;
    int32_t units = 0;
    for (int i = 0; i < n; ++i) {
      const int b = plan.order[c0 + i];
      const int last = last_splits(plan.nsplit, plan.heaviest, last_tile_class(seqs->suffix_len[b], G));
      a.seq[i] = kvt::SeqDesc{b, seqs->prefix_len[b], seqs->suffix_len[b], row_off[b]};
      a.last[i] = (uint8_t)last;
      a.unit_begin[i] = units;
      units += (row_tiles(seqs->suffix_len[b], G) - 1) * plan.nsplit + last;
    }
    a.unit_begin[n] = units;
    const int64_t grid = (int64_t)units * pool->num_kv_heads;
    if (grid > INT32_MAX) return KVT_ERR_INVALID_ARG;
    const hipError_t e = kvt::launch_extend(a, pool->dtype, pool->head_dim, (int)grid, s);
    if (e != hipSuccess) return device_error(e);
  }
  return plan.nsplit > 1 ? combine(a, pool, out, lse, T, num_q_heads, plan.nsplit, plan.heaviest > 0.0, s) : KVT_OK;
}

}  // namespace

extern "C" {

const char* kvt_status_str(kvt_status s) {
  switch (s) {
    case KVT_OK: return "ok";
    case KVT_ERR_INVALID_ARG: return "invalid argument";
    case KVT_ERR_UNSUPPORTED: return "unsupported shape or dtype";
    case KVT_ERR_OUT_OF_RANGE: return "block id out of range or duplicate append target";
    case KVT_ERR_WORKSPACE: return "workspace too small";
    case KVT_ERR_DEVICE: return "HIP launch failed";
    case KVT_ERR_SCRATCH_LIMIT: return "split partials exceed the static scratch (KVT_NOALLOC_SCRATCH_BYTES)";
  }
  return "unknown status";
}

int kvt_last_hip_error(void) { return g_last_hip_error; }

kvt_status kvt_append_kv(const kvt_pool* pool, const kvt_seqs* seqs, const void* k_new, const void* v_new,
                         void* stream) {
  kvt_status st = check_pool(pool);
  if (st != KVT_OK) return st;
  int64_t T = 0;
  if ((st = check_seqs(seqs, &T)) != KVT_OK) return st;
  if (k_new == nullptr || v_new == nullptr || !aligned16(k_new) || !aligned16(v_new)) return KVT_ERR_INVALID_ARG;
  if ((st = check_table_ids(pool, seqs)) != KVT_OK) return st;
  const size_t pool_bytes = (size_t)pool->num_blocks * pool->num_kv_heads * kvt::kBlock * pool->head_dim *
                            elem_bytes(pool->dtype);
  const size_t new_bytes = (size_t)T * pool->num_kv_heads * pool->head_dim * elem_bytes(pool->dtype);
  for (const void* src : {k_new, v_new})
    for (const void* dst : {(const void*)pool->k, (const void*)pool->v})
      if (overlaps(src, new_bytes, dst, pool_bytes)) return KVT_ERR_INVALID_ARG;
  if (seqs->block_table_host != nullptr) {
    // two new tokens may not target one (block, slot)
    std::unordered_set<int64_t> seen;
    seen.reserve((size_t)T * 2);
    for (int b = 0; b < seqs->num_seqs; ++b) {
      const int32_t* row = seqs->block_table_host + (int64_t)b * seqs->max_blocks;
      for (int32_t t = 0; t < seqs->suffix_len[b]; ++t) {
        const int64_t pos = (int64_t)seqs->prefix_len[b] + t;
        const int64_t key = (int64_t)row[pos / kvt::kBlock] * kvt::kBlock + pos % kvt::kBlock;
        if (!seen.insert(key).second) return KVT_ERR_OUT_OF_RANGE;
      }
    }
  }

  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  kvt::AppendArgs a;
  std::memset(&a, 0, sizeof(a));
  a.k_new = k_new;
  a.v_new = v_new;
  a.k_pool = pool->k;
  a.v_pool = pool->v;
  a.block_table = seqs->block_table;
  a.num_blocks = pool->num_blocks;
  a.max_blocks = seqs->max_blocks;
  a.num_kv_heads = pool->num_kv_heads;
  int32_t row = 0;
  for (int b0 = 0; b0 < seqs->num_seqs; b0 += kvt::kSeqsPerLaunch) {
    const int n = std::min(kvt::kSeqsPerLaunch, seqs->num_seqs - b0);
    a.nseq = n;
    a.row_begin = row;
    for (int i = 0; i < n; ++i) {
      const int b = b0 + i;
      a.seq[i] = kvt::SeqDesc{b, seqs->prefix_len[b], seqs->suffix_len[b], row};
      row += seqs->suffix_len[b];
    }
    a.rows = row - a.row_begin;
    const hipError_t e = kvt::launch_append(a, pool->dtype, pool->head_dim, s);
    if (e != hipSuccess) return device_error(e);
  }
  return KVT_OK;
}

size_t kvt_extend_workspace_bytes(const kvt_pool* pool, const kvt_seqs* seqs, int32_t num_q_heads) {
  if (check_pool(pool) != KVT_OK) return 0;
  int64_t T = 0;
  if (check_seqs(seqs, &T) != KVT_OK) return 0;
  if (!heads_ok(pool, num_q_heads, T)) return 0;
  return extend_plan(pool, seqs, num_q_heads, T).ws_bytes;
}

kvt_status kvt_extend_attention(const kvt_pool* pool, const kvt_seqs* seqs, const void* q, int32_t num_q_heads,
                                float scale, void* out, float* lse, void* workspace, size_t workspace_bytes,
                                void* stream) {
  int64_t T = 0;
  const kvt_status st = check_extend(pool, seqs, q, num_q_heads, scale, out, lse, &T);
  if (st != KVT_OK) return st;
  ExtendPlan plan = extend_plan(pool, seqs, num_q_heads, T);
  const kvt_status fit = fit_workspace(&plan, pool, T * num_q_heads, workspace, workspace_bytes);
  if (fit != KVT_OK) return fit;
  return launch_extend_plan(pool, seqs, q, num_q_heads, scale, out, lse, T, plan, workspace, stream);
}

kvt_status kvt_extend_attention_noalloc(const kvt_pool* pool, const kvt_seqs* seqs, const void* q,
                                        int32_t num_q_heads, float scale, void* out, float* lse, void* stream) {
  int64_t T = 0;
  const kvt_status st = check_extend(pool, seqs, q, num_q_heads, scale, out, lse, &T);
  if (st != KVT_OK) return st;
  // the same plan as kvt_extend_attention with a large enough workspace, so
  // both give the same bits, partials in the static scratch; but a call that
  // splits only to fill the chip (its base count is 1) stays unsplit and off
  // the scratch, so that it may overlap other calls on other streams
  ExtendPlan plan = extend_plan(pool, seqs, num_q_heads, T);
  if (plan.nsplit_base == 1) plan.nsplit = 1, plan.heaviest = 0.0;
  void* ws = nullptr;
  if (plan.nsplit > 1) {
    if (plan.ws_bytes > (size_t)KVT_NOALLOC_SCRATCH_BYTES) return KVT_ERR_SCRATCH_LIMIT;
    const hipError_t e = kvt::noalloc_scratch(&ws);
    if (e != hipSuccess) return device_error(e);
  }
  return launch_extend_plan(pool, seqs, q, num_q_heads, scale, out, lse, T, plan, ws, stream);
}

kvt_status kvt_copy_blocks(const kvt_pool* pool, const int32_t* block_ids, const int32_t* block_ids_host,
                           int64_t num_ids, void* host, int32_t direction, void* stream) {
  kvt_status st = check_pool(pool);
  if (st != KVT_OK) return st;
  if (num_ids < 0 || (num_ids > 0 && (block_ids == nullptr || host == nullptr))) return KVT_ERR_INVALID_ARG;
  if (direction != KVT_COPY_TO_HOST && direction != KVT_COPY_TO_DEVICE) return KVT_ERR_INVALID_ARG;
  if (num_ids == 0) return KVT_OK;
  const int64_t page_bytes = (int64_t)pool->num_kv_heads * kvt::kBlock * pool->head_dim * elem_bytes(pool->dtype);
  if (num_ids > (INT64_MAX / 4) / (2 * page_bytes)) return KVT_ERR_INVALID_ARG;
  if (block_ids_host != nullptr) {
    std::unordered_set<int32_t> seen;
    for (int64_t i = 0; i < num_ids; ++i) {
      const int32_t id = block_ids_host[i];
      if (id < 0 || id >= pool->num_blocks) return KVT_ERR_OUT_OF_RANGE;
      // two host pages landing on one pool page would race
      if (direction == KVT_COPY_TO_DEVICE && !seen.insert(id).second) return KVT_ERR_OUT_OF_RANGE;
    }
  }
  // the host side must be pinned memory the device can address
  hipPointerAttribute_t attr;
  std::memset(&attr, 0, sizeof(attr));
  if (hipPointerGetAttributes(&attr, host) != hipSuccess) {
    (void)hipGetLastError();
    return KVT_ERR_INVALID_ARG;
  }
  if (attr.type != hipMemoryTypeHost) return KVT_ERR_INVALID_ARG;
  void* host_dev = attr.devicePointer != nullptr ? attr.devicePointer : host;

  kvt::CopyArgs a;
  a.k_pool = pool->k;
  a.v_pool = pool->v;
  a.ids = block_ids;
  a.n = num_ids;
  a.host = host_dev;
  a.page_bytes = page_bytes;
  a.num_blocks = pool->num_blocks;
  a.to_host = direction == KVT_COPY_TO_HOST ? 1 : 0;
  const int64_t pieces = num_ids * 2 * page_bytes / 16;
  const int grid = (int)std::min<int64_t>((pieces + 255) / 256, 8192);
  const hipError_t e = kvt::launch_copy_blocks(a, grid, reinterpret_cast<hipStream_t>(stream));
  return e == hipSuccess ? KVT_OK : device_error(e);
}

size_t kvt_cascade_workspace_bytes_ex(const kvt_pool* pool, const kvt_seqs* seqs, int32_t shared_len,
                                      int32_t mode, int32_t num_q_heads) {
  if (check_pool(pool) != KVT_OK) return 0;
  int64_t T = 0;
  if (check_seqs(seqs, &T) != KVT_OK) return 0;
  if (!heads_ok(pool, num_q_heads, T)) return 0;
  if (check_shared(seqs, shared_len) != KVT_OK || !mode_ok(mode)) return 0;
  return cascade_plan(pool, seqs, shared_len, num_q_heads, T, mode).ws_bytes;
}

size_t kvt_cascade_workspace_bytes(const kvt_pool* pool, const kvt_seqs* seqs, int32_t shared_len,
                                   int32_t num_q_heads) {
  return kvt_cascade_workspace_bytes_ex(pool, seqs, shared_len, KVT_CASCADE_AUTO, num_q_heads);
}

int32_t kvt_cascade_uses_shared_pass(const kvt_pool* pool, const kvt_seqs* seqs, int32_t shared_len,
                                     int32_t num_q_heads) {
  if (check_pool(pool) != KVT_OK) return -1;
  int64_t T = 0;
  if (check_seqs(seqs, &T) != KVT_OK) return -1;
  if (!heads_ok(pool, num_q_heads, T)) return -1;
  if (check_shared(seqs, shared_len) != KVT_OK) return -1;
  return cascade_plan(pool, seqs, shared_len, num_q_heads, T, KVT_CASCADE_AUTO, true).use_shared ? 1 : 0;
}

kvt_status kvt_cascade_extend_attention(const kvt_pool* pool, const kvt_seqs* seqs, int32_t shared_len,
                                        const void* q, int32_t num_q_heads, float scale, void* out, float* lse,
                                        void* workspace, size_t workspace_bytes, void* stream) {
  return kvt_cascade_extend_attention_ex(pool, seqs, shared_len, KVT_CASCADE_AUTO, q, num_q_heads, scale, out, lse,
                                         workspace, workspace_bytes, stream);
}

kvt_status kvt_cascade_extend_attention_ex(const kvt_pool* pool, const kvt_seqs* seqs, int32_t shared_len,
                                           int32_t mode, const void* q, int32_t num_q_heads, float scale, void* out,
                                           float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  kvt_status st = check_pool(pool);
  if (st != KVT_OK) return st;
  int64_t T = 0;
  if ((st = check_seqs(seqs, &T)) != KVT_OK) return st;
  if ((st = check_shared(seqs, shared_len)) != KVT_OK) return st;
  if (!mode_ok(mode)) return KVT_ERR_INVALID_ARG;
  if (workspace == nullptr && workspace_bytes == 0)   // no scratch: the plain extend computes the same
    return kvt_extend_attention(pool, seqs, q, num_q_heads, scale, out, lse, nullptr, 0, stream);
  if (q == nullptr || out == nullptr) return KVT_ERR_INVALID_ARG;
  if (!heads_ok(pool, num_q_heads, T)) return KVT_ERR_INVALID_ARG;
  if (!(scale > 0.f) || !std::isfinite(scale)) return KVT_ERR_INVALID_ARG;
  if ((st = check_table_ids(pool, seqs)) != KVT_OK) return st;
  if ((st = check_outputs(pool, q, num_q_heads, out, lse, T)) != KVT_OK) return st;
  ExtendPlan plan = cascade_plan(pool, seqs, shared_len, num_q_heads, T, mode);
  if (workspace == nullptr) return KVT_ERR_WORKSPACE;
  if (!plan.use_shared) {
    if ((st = fit_workspace(&plan, pool, T * num_q_heads, workspace, workspace_bytes)) != KVT_OK) return st;
  } else if (workspace_bytes < plan.ws_bytes) {   // room for the base split counts?
    plan = cascade_plan(pool, seqs, shared_len, num_q_heads, T, mode, true);
    if (workspace_bytes < plan.ws_bytes) return KVT_ERR_WORKSPACE;
  }
  if (!aligned16(workspace)) return KVT_ERR_INVALID_ARG;
  if (!plan.use_shared)   // the plain extend is estimated faster: same result, same bits as kvt_extend_attention
    return launch_extend_plan(pool, seqs, q, num_q_heads, scale, out, lse, T, plan, workspace, stream);

  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int G = num_q_heads / pool->num_kv_heads;
  const int nparts = plan.nsplit_shared + plan.nsplit;
  ExtendPlan parts = plan;
  parts.nsplit = nparts;                       // partial buffers: the shared part's splits, then the private ones
  kvt::ExtendArgs a = base_args(pool, seqs, q, num_q_heads, scale, out, lse, T, parts, workspace);
  a.direct = 0;

  // One launch for both parts, the shared part's (longer) units first, so
  // the private parts' units fill the CUs the shared part leaves idle at
  // its end.  Shared part (sequence 0 of the first launch): every new token
  // of the batch against keys [0, shared_len), all of them visible (one
  // virtual sequence whose causal limits start at shared_len - 1), read
  // through the first sequence's table row, with its own key splits.
  // Private parts (the second group): each sequence over keys
  // [shared_len, P_b + i], causal.  Sequences beyond one launch's
  // descriptors go to further launches of private parts only.
  a.nsplit = plan.nsplit_shared;
  a.part_base = 0;
  a.kbeg = 0;
  a.kend = shared_len;
  a.kbeg2 = shared_len;
  a.kend2 = INT32_MAX;
  a.nsplit2 = plan.nsplit;
  a.part_base2 = plan.nsplit_shared;
  std::vector<int32_t> row_off(seqs->num_seqs + 1, 0);
  for (int b = 0; b < seqs->num_seqs; ++b) row_off[b + 1] = row_off[b] + seqs->suffix_len[b];
  size_t c0 = 0;
  for (bool first = true; first || c0 < plan.order.size(); first = false) {
    int n = 0;
    int32_t units = 0;
    if (first) {
      a.seq[0] = kvt::SeqDesc{plan.order[0], shared_len - 1, (int32_t)T, 0};
      a.last[0] = (uint8_t)plan.nsplit_shared;
      a.unit_begin[0] = 0;
      units = row_tiles((int32_t)T, G) * plan.nsplit_shared;
      n = 1;
    }
    a.second = first ? 1 : 0;
    for (; n < kvt::kSeqsPerLaunch && c0 < plan.order.size(); ++n, ++c0) {
      const int b = plan.order[c0];
      a.seq[n] = kvt::SeqDesc{b, seqs->prefix_len[b], seqs->suffix_len[b], row_off[b]};
      a.last[n] = (uint8_t)plan.nsplit;
      a.unit_begin[n] = units;
      units += row_tiles(seqs->suffix_len[b], G) * plan.nsplit;
    }
    a.nseq = n;
    a.unit_begin[n] = units;
    const int64_t grid = (int64_t)units * pool->num_kv_heads;
    if (grid > INT32_MAX) return KVT_ERR_INVALID_ARG;
    const hipError_t e = kvt::launch_extend(a, pool->dtype, pool->head_dim, (int)grid, s);
    if (e != hipSuccess) return device_error(e);
  }
  return combine(a, pool, out, lse, T, num_q_heads, nparts, false, s);
}

size_t kvt_decode_workspace_bytes(const kvt_pool* pool, const kvt_seqs* seqs, int32_t num_q_heads) {
  if (check_pool(pool) != KVT_OK) return 0;
  int64_t T = 0;
  if (check_seqs(seqs, &T) != KVT_OK || T != seqs->num_seqs) return 0;
  if (!heads_ok(pool, num_q_heads, T)) return 0;
  if (num_q_heads / pool->num_kv_heads > kvt::kDecMaxGroup) return 0;
  return make_decode_plan(pool, seqs, num_q_heads).ws_bytes;
}

kvt_status kvt_decode_attention(const kvt_pool* pool, const kvt_seqs* seqs, const void* q, int32_t num_q_heads,
                                float scale, void* out, float* lse, void* workspace, size_t workspace_bytes,
                                void* stream) {
  kvt_status st = check_pool(pool);
  if (st != KVT_OK) return st;
  int64_t T = 0;
  if ((st = check_seqs(seqs, &T)) != KVT_OK) return st;
  if (T != seqs->num_seqs) return KVT_ERR_INVALID_ARG;   // one new token per sequence
  if (q == nullptr || out == nullptr) return KVT_ERR_INVALID_ARG;
  if (!heads_ok(pool, num_q_heads, T)) return KVT_ERR_INVALID_ARG;
  if (num_q_heads / pool->num_kv_heads > kvt::kDecMaxGroup) return KVT_ERR_UNSUPPORTED;
  if (!(scale > 0.f) || !std::isfinite(scale)) return KVT_ERR_INVALID_ARG;
  if ((st = check_table_ids(pool, seqs)) != KVT_OK) return st;
  if ((st = check_outputs(pool, q, num_q_heads, out, lse, T)) != KVT_OK) return st;

  ExtendPlan plan = make_decode_plan(pool, seqs, num_q_heads);
  if ((st = fit_workspace(&plan, pool, T * num_q_heads, workspace, workspace_bytes)) != KVT_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int per_cu = decode_per_cu(pool, seqs, plan);
  kvt::ExtendArgs a = base_args(pool, seqs, q, num_q_heads, scale, out, lse, T, plan, workspace);
  for (size_t c0 = 0; c0 < plan.order.size(); c0 += kvt::kSeqsPerLaunch) {
    const int n = (int)std::min<size_t>(kvt::kSeqsPerLaunch, plan.order.size() - c0);
    a.nseq = n;
    for (int i = 0; i < n; ++i) {
      const int b = plan.order[c0 + i];
      a.seq[i] = kvt::SeqDesc{b, seqs->prefix_len[b], 1, b};   // row of sequence b is b
      a.unit_begin[i] = i * plan.nsplit;
    }
    a.unit_begin[n] = n * plan.nsplit;
    const int64_t grid = (int64_t)n * plan.nsplit * pool->num_kv_heads;
    const hipError_t e = kvt::launch_decode(a, pool->dtype, pool->head_dim, (int)grid, per_cu, s);
    if (e != hipSuccess) return device_error(e);
  }
  return plan.nsplit > 1 ? combine(a, pool, out, lse, T, num_q_heads, plan.nsplit, false, s) : KVT_OK;
}

}  // extern "C"
