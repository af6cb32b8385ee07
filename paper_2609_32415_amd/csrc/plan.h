// Work decomposition of an attention launch: host arithmetic on sizes and on what the device
// holds at once, without a device call, so that it can be checked on the CPU.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "internal.h"

namespace refadapt {

// ---- bf16: whole query tiles and key chunks
//
// All query tiles of a launch cost the same (each attends to every key tile),
// so the resident workgroups (slots = CUs x workgroups per CU) run them in
// rounds. Cost model in units of "one key tile processed by every resident
// workgroup": a round of items of L key tiles costs L, or kLoneRound * L when
// the round holds no more items than there are CUs (a workgroup alone on its
// CU runs faster); a chunk adds a fixed start-up and drain of kChunkOverhead
// key tiles; the merge costs its partial-result traffic. The plan keeps the
// largest number of whole rounds and splits only the remainder (plus, when it
// pays, one more round) into chunks of at least kMinChunk key tiles.
constexpr int kMinChunk = 4;
constexpr double kChunkOverhead = 2.0;
constexpr double kLoneRound = 0.67;
constexpr int kMaxChunks = 32;

inline SplitPlan whole_plan(int64_t tiles) { return SplitPlan{(int32_t)tiles, 0, 1, (int32_t)tiles}; }

// Cost of running `items` items of `len` key tiles each in rounds of `slots`.
inline double rounds_cost(int64_t items, double len, int64_t slots, int64_t cus) {
  const int64_t full = items / slots, last = items - full * slots;
  return full * len + (last == 0 ? 0.0 : last > cus ? len : kLoneRound * len);
}

inline SplitPlan plan_split(int64_t tiles, int nt, AttnSlots sl, int head_dim, int bm) {
  SplitPlan best = whole_plan(tiles);
  const int64_t slots = (int64_t)sl.cus * sl.per_cu;
  if (tiles <= 0 || slots <= 0 || nt < 2 * kMinChunk) return best;
  // A split must beat whole tiles by 3%; among splits the cheapest wins.
  double best_cost = 0.97 * rounds_cost(tiles, nt, slots, sl.cus);
  // Seconds for every resident workgroup to process one key tile (~1 PFLOP/s of
  // attention) and to move one split item's partial rows twice (~4 TB/s).
  const double tile_s = slots * 4.0 * bm * kAttnBf16BN * head_dim / 1.0e15;
  const double item_s = 2.0 * bm * (head_dim + 4) * 4.0 / 4.0e12;
  for (int extra = 0; extra < 2; ++extra) {
    const int64_t rem = tiles % slots + (int64_t)extra * slots;
    if (rem == 0 || rem > tiles) continue;
    const int64_t rounds = (tiles - rem) / slots;
    for (int c = 2; c <= kMaxChunks && c * kMinChunk <= nt; ++c) {
      const int64_t items = rem * c;
      if (items > 2 * slots) break;
      const int chunk = (nt + c - 1) / c;
      const double cost = (double)rounds * nt + rounds_cost(items, chunk + kChunkOverhead, slots, sl.cus) +
                          (items * item_s + 5e-6) / tile_s;
      if (cost < best_cost) {
        best_cost = cost;
        best = SplitPlan{(int32_t)(tiles - rem), (int32_t)rem, c, (int32_t)(tiles - rem + items)};
      }
    }
  }
  return best;
}

// Estimated time (us) of a plan on workgroups of bm query rows, to choose between the two
// workgroup sizes. (plan_split compares chunk counts on one size, where its units cancel; here the
// two sizes' rates have to be right against each other.) Time of one key tile in a round, measured per head dim with few workgroups
// (one a CU at most, `lone`) and with a full round (`full`): 256-row workgroups keep a CU to
// themselves and share a K/V tile between eight wavefronts; 128-row ones run two a CU, or one at
// less time a tile, for twice the K/V traffic.
struct TileTime {
  double lone, full;
};
constexpr double kStartTiles = 2.0;  // start-up and drain of a workgroup, in key tiles
constexpr double kMergeUs = 5.0;     // the merge's launch; its traffic is charged by bytes

inline TileTime tile_time(int head_dim, int bm) {
  if (bm == kAttnBf16BM) return head_dim == 128 ? TileTime{1.27, 1.62} : TileTime{1.02, 1.07};
  return head_dim == 128 ? TileTime{0.95, 1.70} : TileTime{0.80, 1.06};
}

inline double plan_us(const SplitPlan& pl, int nt, AttnSlots sl, int head_dim, int bm) {
  const TileTime tt = tile_time(head_dim, bm);
  const int64_t cus = sl.cus, slots = cus * sl.per_cu;
  const auto rounds = [&](int64_t items, double len) {
    const int64_t full = items / slots, last = items - full * slots;
    // A partly filled last round draws less power and runs at a higher clock: from `lone` with few
    // workgroups to `full`, or, with one 128-row workgroup a CU, to 0.2 us above `lone` (fitted, as
    // the rates, to the launches named at prefers_small).
    const double top = bm == kAttnBf16BM ? tt.full : tt.lone + 0.2;
    const double part = last > cus ? tt.full : last > 0 ? tt.lone + (top - tt.lone) * (double)last / (double)cus : 0.0;
    return len * ((double)full * tt.full + part);
  };
  double us = rounds(pl.whole, nt + kStartTiles);
  if (pl.split_tiles > 0) {
    const int64_t items = (int64_t)pl.split_tiles * pl.chunks;
    us += rounds(items, (nt + pl.chunks - 1) / pl.chunks + kStartTiles) + kMergeUs +
          (double)items * 2.0 * bm * (head_dim + 4) * 4.0 / 4.0e6;
  }
  return us;
}

// A launch's sizes and what the device holds at once of each workgroup size.
struct PlanShape {
  int64_t bh;
  int32_t head_dim, n_ref, n_tgt;
  AttnSlots big, small;  // workgroups of kAttnBf16BM and of kAttnBf16SmallBM rows
};

// Plan of one query set (target rows, or reference rows too) on tiles of bm rows, and the
// workspace bytes that its split items need.
struct QueryPlan {
  SplitPlan plan;
  int64_t qt_ref, qt_tgt;
  int64_t items;  // split items
  int bm;         // query rows per tile
  double us;      // estimated time, 0 when the device cannot be queried
};

inline size_t part_o_bytes(int64_t items, int bm, int head_dim) {
  return (size_t)items * bm * head_dim * sizeof(float);
}
inline size_t items_ws_bytes(int64_t items, int bm, int head_dim) {
  return items > 0 ? part_o_bytes(items, bm, head_dim) + (size_t)items * bm * 5 * sizeof(float) : 0;
}

inline QueryPlan plan_queries_bm(const PlanShape& s, bool ref_queries, bool split, int bm) {
  QueryPlan q{};
  q.bm = bm;
  q.qt_ref = ref_queries && s.n_ref > 0 ? ((int64_t)s.n_ref + bm - 1) / bm : 0;
  q.qt_tgt = ((int64_t)s.n_tgt + bm - 1) / bm;
  const int64_t tiles = s.bh * (q.qt_ref + q.qt_tgt);
  q.plan = whole_plan(tiles);
  if (tiles > 0x7fffffff) return q;
  const AttnSlots slots = bm == kAttnBf16BM ? s.big : s.small;
  const int nt = (s.n_ref + kAttnBf16BN - 1) / kAttnBf16BN + (s.n_tgt + kAttnBf16BN - 1) / kAttnBf16BN;
  if (split) q.plan = plan_split(tiles, nt, slots, s.head_dim, bm);
  q.items = (int64_t)q.plan.split_tiles * q.plan.chunks;
  if (slots.cus > 0) q.us = plan_us(q.plan, nt, slots, s.head_dim, bm);
  return q;
}

// What a launch of one K/V mode runs: the query sets it may hold (a device-decided launch both).
struct LaunchMode {
  bool all, tgt;  // reference and target rows; target rows alone
  bool seg;       // reference segments
};

// The two query sets on both workgroup sizes.
struct LaunchPlans {
  QueryPlan tgt[2], all[2];  // [0]: 256 rows, [1]: 128 rows
  bool split;                // key ranges may be split

  // A launch runs workgroups of 128 query rows where the estimates say by more than their own error
  // (3 to 5%) that these are faster, else of 256: launches of few tiles, which leave CUs idle or one
  // workgroup each. Measured, us, 256 against 128 rows: 4 heads, 300 + 256 tokens, all queries
  // 21.8 / 15.9; 24 heads, 1024 target queries over 2048 keys 43.6 / 38.3; 12 heads, 700 + 800, all
  // 40.8 / 30.5; 24 heads, 2095 + 1009, all 133 / 135; 24 heads, 4352 + 4096, all 755 / 778. The
  // segment kernel runs 256 rows only.
  // Where key ranges may be split the estimates are those of the target queries and of all queries
  // together (3% each), so that the choice is the same for both, wherever the K/V come from
  // and whoever decides: a device-decided launch gives the bits of the explicit launch of the same
  // queries. (Over 44 shapes of 1 to 48 heads and 64 to 8192 tokens explicit launches of all and of
  // target queries take 0.99 and 0.98, device-decided ones 0.99 and 0.97 of the time with a choice
  // per mode.) Whole rows are summed in the same order on both sizes: without splits the launch's
  // own sets count (24 heads of 64, 1500 + 700, all queries 41.8 us; 45.0 by both sets).
  bool prefers_small(LaunchMode m) const {
    double big = split ? 0.97 * 0.97 : 0.95, small = 1.0;
    if (split || m.tgt) big *= tgt[0].us, small *= tgt[1].us;
    if (split || m.all) big *= all[0].us, small *= all[1].us;
    return !m.seg && small > 0.0 && small < big;
  }
  // Workspace of the launch's split items on one workgroup size.
  size_t ws_bytes(int size, LaunchMode m, int head_dim) const {
    const int64_t items = std::max(m.all ? all[size].items : 0, m.tgt ? tgt[size].items : 0);
    return items_ws_bytes(items, tgt[size].bm, head_dim);
  }
};

inline LaunchPlans plan_launch(const PlanShape& s, bool split) {
  LaunchPlans l;
  l.split = split;
  for (int i = 0; i < 2; ++i) {
    const int bm = i == 0 ? kAttnBf16BM : kAttnBf16SmallBM;
    l.tgt[i] = plan_queries_bm(s, false, split, bm);
    l.all[i] = s.n_ref > 0 ? plan_queries_bm(s, true, split, bm) : l.tgt[i];
  }
  return l;
}

// Workspace to ask for, the same for every K/V source of the query sets: what the plan needs that a
// launch without segments prefers, or the one on 256 rows where that is more, with which it runs too.
inline size_t launch_ws_bytes(const LaunchPlans& l, LaunchMode m, int head_dim) {
  const size_t big = l.ws_bytes(0, m, head_dim);
  return l.prefers_small({m.all, m.tgt, false}) ? std::max(big, l.ws_bytes(1, m, head_dim)) : big;
}

// Workspace with which a launch with per-segment masses splits key ranges: that of the launch
// without them and one log-sum-exp per segment of each partial row; 0 when its plan splits nothing.
inline size_t launch_seg_ws_bytes(const LaunchPlans& l, LaunchMode m, int head_dim, int n_seg) {
  const QueryPlan& q = m.all ? l.all[0] : l.tgt[0];
  return q.items > 0 ? launch_ws_bytes(l, m, head_dim) + (size_t)q.items * q.bm * n_seg * sizeof(float) : 0;
}

// The workgroup size (index) of a launch with a workspace of ws_bytes: the preferred one if its
// partials fit.
inline int launch_size(const LaunchPlans& l, LaunchMode m, int head_dim, size_t ws_bytes) {
  return l.prefers_small(m) && l.ws_bytes(1, m, head_dim) <= ws_bytes ? 1 : 0;
}

// ---- fp32: query subtiles per workgroup and key groups inside it
//
// Every workgroup of QW query subtiles costs QW units of work, so a
// launch of W workgroups takes about ceil(W / CUs) * QW units of the slower CUs' time: few
// subtiles per workgroup (and so more key groups) spread a small launch over more CUs and waste
// less of the last round, many share a K/V tile between more wavefronts. `lone` and `full` are
// the measured time per unit of each shape with one workgroup on a CU and with several, relative
// to (QW 4, several): 16.5 ns per key at head dim 128.
//   us, shapes QW 4 / 2 / 1:  24 heads, 1101 + 1024, all queries 584 / 600 / 602; target queries
//   296 / 274 / 285; 48 heads of 64, 2000 + 1900, target 829 / 887 / 962; 8 heads, 2048 + 2048, all
//   558 / 629 / 705; 6 heads, 700 + 500, all 101 / 66 / 70; 2 heads, 2000 + 100, target
//   171 / 107 / 54; 2 heads of 64, 256 + 256, all 28 / 20 / 12.
// The first launch takes QW 2: counting whole rounds charges QW 4's 384 target workgroups two,
// though two share a CU, and the estimates (128 / 103 / 122) are further apart than the times; QW 2
// is 3% slower than QW 4 there on all queries and 7% faster on the target ones. Fewer keys per sum
// also mean a smaller error: 9.2e-7 / 7.2e-7 / 5.9e-7 there.
// The choice weighs the launch with and without the reference queries alike and does not depend
// on which of the two this is, so target rows are summed in the same order in both.
struct F32Cost {
  int subtiles;
  double lone, full;
};
constexpr F32Cost kF32Costs[] = {{4, 1.18, 1.0}, {2, 1.45, 1.11}, {1, 1.57, 1.25}};
constexpr int kLongKeys = 512;

struct F32Split {
  int subtiles;    // query subtiles of 16 rows per workgroup
  int wavefronts;  // of which subtiles share each key group
};

inline F32Split f32_split(int64_t bh, int32_t n_ref, int32_t n_tgt, int64_t cus) {
  F32Split best{4, 4};
  double best_cost = 0.0;
  for (const F32Cost& s : kF32Costs) {
    const int64_t bq = 16 * s.subtiles;
    const int64_t tgt = bh * ((n_tgt + bq - 1) / bq), all = tgt + bh * ((n_ref + bq - 1) / bq);
    double cost = 1.0;
    for (const int64_t w : {tgt, all})
      cost *= (double)((w + cus - 1) / cus * s.subtiles) * (w <= cus ? s.lone : s.full);
    if (best_cost == 0.0 || cost < best_cost) {
      best.subtiles = s.subtiles;
      best_cost = cost;
    }
  }
  // One subtile per workgroup: four key groups, or eight where the launch leaves the CUs one
  // workgroup each and the groups still have several key tiles (2 heads, 2000 + 100 keys 54
  // against 58 us, one head of 64 with 2048 + 2048 keys 57 against 68; 64 + 64 keys 9.5 against 8.1).
  if (best.subtiles == 1 && bh * ((n_tgt + 15) / 16) <= cus && (int64_t)n_ref + n_tgt >= kLongKeys) best.wavefronts = 8;
  return best;
}

}  // namespace refadapt
