// Host-side plan builder (paper Section 3.2: plans are generated per batch before the data
// plane runs; Section 4.3: segments near the root of the prefix tree are hot, so requests
// that share a run of segments are batched against it).
//
// Every request's list is walked down the pool's prefix tree (nodes are made as needed and stay
// for later batches; each node on the way takes the request's new tokens as load).  A maximal
// chain of tree nodes that the same set of requests passes through becomes one work item whose
// query rows are all new tokens of those requests.  Items with few rows per kv head are cut into
// split-K chunks.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <new>
#include <numeric>
#include <queue>
#include <unordered_set>

#include "tl_internal.h"

using namespace tl;

namespace {

struct RawItem {
  std::vector<int32_t> reqs;   // ascending
  int32_t src_req;             // request whose list supplies the run
  int32_t begin, end;          // list positions [begin, end)
};

// The split-K units of a batch.
struct UnitLoad {
  int64_t units = 0, tokens = 0, longest = 0;      // kv tokens of all units and of the longest

  bool even() const { return 10 * tokens >= 7 * units * longest; }
};

// kv heads per workgroup of the split-K kernel: the most of 8, 4, 2 or 1 that divides kv_heads (whole
// token rows per workgroup stream best), halved while the launch stays one round of the CUs: then a unit's heads
// go to several workgroups, whose waves share the unit's tokens.  Measured, a workgroup per unit with one wave per head
// against this deal: 64 requests of a one-kv-head layer 391 -> 123 us (1.8 -> 5.8 TB/s; seven of eight waves had no
// head), one request of 15.9k tokens with 8 kv heads 34 -> 15 us (32 workgroups became 256); with 8 heads and 200 units
// or more the two are the same launch (234 us, 5.97 TB/s; 811 units 3.83 ms, 6.0 TB/s).
// More than half a round of units of one length is left alone, a thin second round costs more than the first
// gains (168 units of 512 tokens, 8 heads: 55.9 us, halved 62.6); units of uneven length are halved up to three
// quarters of a round, the shorter ones then fill the second (131 units of up to 512 tokens 35.7, halved 33.9).
// Where 8 does not divide the heads, 8 to a workgroup with some waves idle (at most 7 of 16) is better for one round of even
// units that dealt by a divisor would be more (227 units of 5 heads: 92 us, 102 with a workgroup per head; 118 of 12 heads
// 58 and 61, of 9 heads 47 and 55; but 196 uneven units of 5 heads 190 and 156, and 64 of 12 heads, a round either way, 31.5 and 26.7).
int32_t plan_unit_heads_log2(int32_t kv_heads, const UnitLoad& load, int64_t n_cu) {
  int32_t log2 = 3;
  while (kv_heads & ((1 << log2) - 1)) --log2;
  const int32_t eights = unit_head_blocks(kv_heads, 3);
  if (kv_heads % 8 && 2 * kv_heads >= 9 * eights && load.even() && 8 * load.units * eights > 3 * n_cu && load.units * eights <= n_cu &&
      load.units * unit_head_blocks(kv_heads, log2) > n_cu)
    return 3;
  while (log2 > 0 && 2 * load.units * unit_head_blocks(kv_heads, log2) <= n_cu) --log2;
  if (log2 > 0 && !load.even() && 4 * load.units * unit_head_blocks(kv_heads, log2) < 3 * n_cu) --log2;
  return log2;
}

// What a batch costs, in KV tiles of a row-tile workgroup (1.5 us): a workgroup's start, first loads and epilogue;
// the launch of one-pass rows behind the split-K units', and the causal launch and merge of the three steps; bytes of
// partials and of split-K units in the time of a tile.  Fitted to 758 random batches of 1 to 12 prefill chunks beside 2 to
// 250 decoded tokens in eight layer shapes, 37 us to 3.2 ms, each timed both as one-pass rows and on the three
// steps; the two estimates are off by 12 and 16 % in the root mean square.
constexpr int64_t kTileStart = 5;
constexpr double kOnePassLaunch = 8, kThreeStepLaunches = 6;
constexpr double kBytesPerTile = 7.8e6, kUnitBytesPerTile = 9.75e6;

// KV tiles from which a list is cut where its launch ends unevenly, so that a piece's start stays small: the pieces are
// even, so half of it (1024 tokens) is the shortest.  (At least this much a piece instead: 4 chunks of 64 to 364 tokens on
// 1.4k to 11k beside 27 decoded tokens 246 us for 235.)
constexpr int32_t kMinPieceTiles = 2048 / kKvTile;
constexpr int64_t kShortPieceTiles = 512 / kKvTile;      // the shortest piece where the launch leaves CUs idle (one_round_cut)

// Partial rows of `row_tiles` row tiles, written and read.
double merge_tiles(int64_t row_tiles, int32_t kv_heads) {
  return (double)row_tiles * kRowTile * kv_heads * (2 * 4 * kHeadDim) / kBytesPerTile;
}

// A launch of split-K units and row tiles together, both given as launches of their own.  Row tiles fill the CUs that
// the units' last round of workgroups leaves idle (up to half of them: they are as long as their lists), and some
// of what either waits for beside that.
double joint_tiles(double units, int64_t unit_blocks, double tiles, int64_t n_cu) {
  const int64_t room = (unit_blocks + n_cu - 1) / n_cu * n_cu;
  const double idle = units * (double)(room - unit_blocks) / (double)room, shorter = std::min(units, tiles);
  return units + tiles - std::min(shorter, std::min(idle, 0.5 * tiles) + 0.25 * shorter);
}

// When a launch of split-K units and row tiles ends (us) whose units are taken by `lanes` workgroups in turn: a walk from end
// to end of a workgroup over the launch, as it is dealt.  An XCD takes every eighth workgroup, in order, as its CUs fall free;
// walked are the first, which stands for those with a unit workgroup more, and the last (all eight: 45 of the batches below
// more than 1.02 for 54, and a plan of 196 units and 656 row tiles takes 330 us for 223).  A unit's workgroup streams
// kUnitRate at most, all of them share what row tiles leave of HBM; a row tile's takes its KV tiles from HBM, with the others
// of its list from L2, and is slower the more of HBM is asked for and the more of the chip multiplies (power).  Fitted to
// tl_segment_attn of 12774 random batches of 1 to 8 prefill chunks beside 4 to 200 decoded tokens, each timed with all units
// at once and with two in turn: the ratio of the two ends is off by 6.5 % in the root mean square.
constexpr int64_t kXcds = 8;
constexpr double kHbmRate = 5.9e6, kUnitRate = 47e3, kRowTileRate = 42e3;      // bytes per us: of HBM, of a unit's workgroup, of a row tile's by itself
constexpr double kUnitStart = 4.0;                                              // us: a unit's start and end
constexpr double kRowTileUs = 1.1, kRowTileHbmUs = 0.5, kRowTilePowerUs = 0.4;  // us of a KV tile, and what HBM load and a full chip add
double joint_end(const std::vector<double>& unit_bytes, int64_t head_blocks, int64_t lanes, const std::vector<Work>& tiles,
                 const std::vector<double>& tile_rate, int32_t kv_heads, int64_t n_cu) {
  struct End {
    double at, rate;       // in bytes that each unit's, in KV tiles that each row tile's workgroup has seen go by since the start
    int xcd;
    bool operator<(const End& o) const { return at > o.at; }
  };
  const int64_t n_units = (int64_t)unit_bytes.size(), n = n_units * head_blocks, row0 = (lanes + kXcds - 1) / kXcds * kXcds;
  const int64_t total = row0 + (int64_t)tiles.size() * kv_heads, cus = std::max<int64_t>(1, n_cu / kXcds);
  const double hbm = kHbmRate * (double)(cus * kXcds) / kComputeUnits;
  std::priority_queue<End> units, rows;
  const int64_t more = lanes % kXcds ? lanes % kXcds : kXcds / 2;
  const double weight[2] = {(double)more, (double)(kXcds - more)};
  double t = 0, bytes = 0, kv = 0, row_rate = 0, n_at_units = 0, n_at_rows = 0;
  int64_t next[2] = {0, kXcds - 1}, idle[2] = {cus, cus};
  auto deal = [&](int x) {
    for (; idle[x] > 0 && next[x] < total; next[x] += kXcds) {
      const int64_t wg = next[x];
      if (wg >= lanes && wg < row0) continue;
      --idle[x];
      if (wg < lanes) {
        double chain = 0;
        for (int64_t first = 0; first < n; first += lanes) {
          const int64_t i = (first / lanes) & 1 ? first + lanes - 1 - wg : first + wg;
          if (i < n) chain += unit_bytes[i % n_units] + kUnitStart * kUnitRate;
        }
        units.push(End{bytes + chain, 0, x});
        n_at_units += weight[x];
      } else {
        const int64_t tile = (wg - row0) / kv_heads;
        rows.push(End{kv + (double)(tiles[tile].n_full + tiles[tile].n_part + kTileStart), tile_rate[tile], x});
        row_rate += weight[x] * tile_rate[tile];
        n_at_rows += weight[x];
      }
    }
  };
  deal(0);
  deal(1);
  while (!units.empty() || !rows.empty()) {
    const double left = std::max(hbm - row_rate, 0.2 * hbm), asked = kUnitRate * n_at_units, busy = n_at_rows / (double)(cus * kXcds);
    const double per_unit = asked > left ? kUnitRate * left / asked : kUnitRate;
    const double per_row = 1 / (kRowTileUs + kRowTileHbmUs * std::min(1.0, asked / left) + kRowTilePowerUs * busy * busy * busy);
    const double unit_end = units.empty() ? HUGE_VAL : (units.top().at - bytes) / per_unit, row_end = rows.empty() ? HUGE_VAL : (rows.top().at - kv) / per_row;
    const double dt = std::min(unit_end, row_end);
    t += dt;
    bytes = unit_end <= row_end ? units.top().at : bytes + dt * per_unit;
    kv = row_end <= unit_end ? rows.top().at : kv + dt * per_row;
    for (; !units.empty() && units.top().at <= bytes; units.pop()) {
      ++idle[units.top().xcd];
      n_at_units -= weight[units.top().xcd];
    }
    for (; !rows.empty() && rows.top().at <= kv; rows.pop()) {
      ++idle[rows.top().xcd];
      n_at_rows -= weight[rows.top().xcd];
      row_rate -= weight[rows.top().xcd] * rows.top().rate;
    }
    deal(0);
    deal(1);
  }
  return t;
}

// Workgroups that take the split-K units beside row tiles.  All units at once keep HBM busy and leave row tiles the few CUs that are
// over; with half as many workgroups that take two units each in turn, row tiles and units may run side by side for longer,
// or the units may be what ends last: whichever the walk says ends earlier, two in turn by a margin of 3 % and 3 us.  Of the 12774
// batches 3030 are taken in turn: 0.88 of the time of all at once in the mean, 54 of them more than 1.02 and 12 more than 1.05;
// of 14546 others, which nothing was fitted to, 2515: 0.90, 39 and 8, 1.12 at most.  Over the 12774 0.971 of all at once, and
// the better of the two each time would be 0.959.  (Lines on the ratio of units to row tiles and on rounds of either take 1678,
// 71 of them more than 1.02 and 38 more than 1.05, up to 1.29: over all 0.988.  The walk passes by 440 that gained 2 % or more there.)
// Not where several workgroups share a unit with eight heads each (16 kv heads): at once they read the parts of a token's row
// together, in turn one after the other (180 batches where the walk says 0.92 or less 0.99, 35 of them more than 1.02).
// Three in turn: 1.01 in the mean.
int64_t plan_unit_lanes(const std::vector<double>& unit_bytes, int32_t heads_log2, const std::vector<Work>& tiles, int32_t kv_heads, int64_t n_cu) {
  const int64_t head_blocks = unit_head_blocks(kv_heads, heads_log2), all = (int64_t)unit_bytes.size() * head_blocks, half = (all + 1) / 2;
  // (row tiles in more than 16 rounds of the CUs leave no gaps that a walk would find)
  if (unit_bytes.empty() || tiles.empty() || n_cu <= 0 || (head_blocks > 1 && heads_log2 == 3) || (int64_t)tiles.size() * kv_heads > 16 * n_cu) return all;
  std::vector<double> tile_rate(tiles.size());
  for (size_t first = 0, end; first < tiles.size(); first = end) {       // the row tiles of an item, up to eight of them at a time
    for (end = first; end < tiles.size() && tiles[end].kv_off == tiles[first].kv_off;) ++end;
    for (size_t i = first; i < end; ++i) tile_rate[i] = kRowTileRate / (double)std::min<size_t>(end - first, 8);
  }
  const double at_once = joint_end(unit_bytes, head_blocks, all, tiles, tile_rate, kv_heads, n_cu);
  return joint_end(unit_bytes, head_blocks, half, tiles, tile_rate, kv_heads, n_cu) < 0.97 * at_once - 3 ? half : all;
}

struct RowWork {
  int64_t kv_tiles, row_tiles;
};

// KV tiles until the last of `lanes` CUs is done when they take `work` (kv_tiles + kTileStart for each row
// tile) longest first; with many more row tiles than CUs, which leave no gaps, the mean.
int64_t makespan(std::vector<RowWork> work, int64_t lanes) {
  int64_t total = 0, longest = 0, n = 0;
  for (const RowWork& w : work) {
    total += (w.kv_tiles + kTileStart) * w.row_tiles;
    longest = std::max(longest, w.kv_tiles + kTileStart);
    n += w.row_tiles;
  }
  if (n > 16 * lanes) return std::max(longest, total / lanes);
  std::sort(work.begin(), work.end(), [](const RowWork& a, const RowWork& b) { return a.kv_tiles > b.kv_tiles; });
  std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> busy;
  int64_t end = 0;
  for (const RowWork& w : work)
    for (int64_t i = 0; i < w.row_tiles; ++i) {
      int64_t at = 0;
      if ((int64_t)busy.size() >= lanes) {
        at = busy.top();
        busy.pop();
      }
      busy.push(at + w.kv_tiles + kTileStart);
      end = std::max(end, at + w.kv_tiles + kTileStart);
    }
  return end;
}

// What a work item over a run of a list walks: slots (a repeated one once), their tokens and KV tiles.
struct Walk {
  int32_t slots;
  int64_t tokens, kv_tiles;
};

struct RowItem {       // a work item of row tiles
  Walk walk;
  int64_t row_tiles, halves;      // workgroups per kv head and piece, whole and where each takes half the rows
  int64_t rows;                   // per kv head
};

// How the lists of a launch's row-tile items are cut along the KV: into `chunks` pieces of min_slots or more, or
// into pieces of about `longest` KV tiles (0: not cut).
struct RowCut {
  int32_t chunks = 1, min_slots = 1;
  int64_t longest = 0;

  // slots per piece; the last piece takes what is left
  int32_t step(const Walk& w) const {
    if (chunks > 1) return std::max(min_slots, (w.slots + chunks - 1) / chunks);
    if (longest == 0) return w.slots;
    const int64_t n = std::max<int64_t>(1, std::min((w.kv_tiles + longest - 1) / longest, w.kv_tiles / kShortPieceTiles));
    return (int32_t)((w.slots + n - 1) / n);
  }
};

// The row tiles of the items' pieces, and the partial rows that they write (x kRowTile).
int64_t cut_items(const std::vector<RowItem>& items, const RowCut& cut, std::vector<RowWork>& pieces) {
  int64_t n_partial = 0;
  pieces.clear();
  for (const RowItem& it : items) {
    if (it.walk.slots == 0) continue;
    const int64_t step = std::min(cut.step(it.walk), it.walk.slots), whole = it.walk.slots / step, rest = it.walk.slots % step;
    const int64_t kv = (it.walk.kv_tiles * step + it.walk.slots - 1) / it.walk.slots;
    pieces.push_back(RowWork{kv, whole * it.row_tiles});
    if (rest > 0) pieces.push_back(RowWork{std::max<int64_t>(1, it.walk.kv_tiles - kv * whole), it.row_tiles});
    n_partial += (whole + (rest > 0)) * it.row_tiles;
  }
  return n_partial;
}

// Workgroups of the items' pieces; `halves`: where a row tile of more than half its rows is two.
int64_t cut_workgroups(const std::vector<RowItem>& items, const RowCut& cut, int32_t kv_heads, bool halves) {
  int64_t wgs = 0;
  for (const RowItem& it : items) {
    if (it.walk.slots == 0) continue;
    const int64_t step = cut.step(it.walk);
    wgs += (it.walk.slots + step - 1) / step * (halves ? it.halves : it.row_tiles) * kv_heads;
  }
  return wgs;
}

// Row tiles as two workgroups of half the rows each where that stays one round of the CUs: the four waves of a half have a
// SIMD each, and a tile takes 0.76 us instead of 1.12.  (3 chunks of 256 tokens with 8 kv heads, 96 workgroups: pool
// launch 15.5 -> 13.4 us, causal launch 13.4 -> 11.4; one of 322 to 645 as one-pass rows 25.8 -> 20.9.)  A second half
// without rows ends at once but holds a CU until then: where they do not all fit beside the others an eighth of the round is left for
// them (17 row tiles of 8 kv heads of which 15 have two halves, 256 of 272 workgroups: 41.6 us whole, 47.7 halved), and
// no more than two in five of the row tiles have two halves (18 of 8 kv heads, every other one narrow, 216 of 288 workgroups:
// some second halves wait for a whole chain, 63.7 us; up to 1.4 workgroups a row tile nothing waits, from 1.5 on 4 us in the mean).
// `wgs`: with two for a tile of more than half its rows.
bool halves_fit(int64_t row_tiles, int64_t wgs, int32_t kv_heads, int64_t n_cu) {
  return wgs > row_tiles && (2 * row_tiles * kv_heads <= n_cu || (8 * wgs * kv_heads <= 7 * n_cu && 5 * wgs <= 7 * row_tiles));
}

// What the three steps of a launch of one round take (us), but for what is the same however its lists are cut: the longest
// chain of tiles, workgroups that start, partials written and read.  Fitted to 4508 random batches, each timed in five
// cuts: differences between the cuts of a batch are off by 1.9 us in the root mean square.
double one_round_us(const std::vector<RowItem>& items, const RowCut& cut, int64_t n_cu, int32_t kv_heads, bool wide) {
  int64_t row_tiles = 0, wgs = 0, rows = 0, chain = 0;
  for (const RowItem& it : items) {
    if (it.walk.slots == 0) continue;
    const int64_t step = std::min(cut.step(it.walk), it.walk.slots), n = (it.walk.slots + step - 1) / step;
    row_tiles += n * it.row_tiles;
    wgs += n * it.halves;
    rows += n * it.rows;
    chain = std::max(chain, (it.walk.kv_tiles * step + it.walk.slots - 1) / it.walk.slots);
  }
  const double tile = wide && !halves_fit(row_tiles, wgs, kv_heads, n_cu) ? 1.0 : 0.68;
  return tile * (double)chain + 7.4 * (double)(row_tiles * kv_heads) / (double)n_cu + 0.2e-6 * (double)(rows * kv_heads) * (4 * kHeadDim);
}

// A launch that leaves CUs idle where its lists are cut into pieces of 2048 tokens (half of the CUs, or where row tiles have half
// their rows or less, which are bound by their chain of tiles alone, any) waits for the longest chain of
// tiles: pieces down to 512 tokens, no more than one round of whole row tiles, as one_round_us has it.
// Of 3118 other batches, three steps, against pieces of 2048 tokens: 0.80 of the time in the mean, 72 more than 1.02 (the shortest
// pieces that are one round, partials not counted: 0.81, 179 of them).
RowCut one_round_cut(const std::vector<RowItem>& items, int64_t n_cu, int32_t kv_heads, const RowCut& otherwise) {
  bool wide = false;
  for (const RowItem& it : items) wide = wide || it.halves > it.row_tiles;
  RowCut best = otherwise;
  double best_us = one_round_us(items, otherwise, n_cu, kv_heads, wide);
  RowCut c;
  for (c.longest = kShortPieceTiles; c.longest < kMinPieceTiles; c.longest += kShortPieceTiles / 4) {
    if (cut_workgroups(items, c, kv_heads, false) > n_cu) continue;
    const double us = one_round_us(items, c, n_cu, kv_heads, wide);
    if (us < best_us) {
      best_us = us;
      best = c;
    }
  }
  return best;
}

// Row-tile items of a small batch: when all row tiles together are fewer workgroups than the
// GPU has CUs, long slot lists are cut into chunks (each a work item with partial rows of its
// own, merged like any other) until there are about two workgroups per CU; a chunk keeps at
// least 2048 tokens so that its start-up stays small against its work.  With more row tiles than that,
// lists longer than half the mean load of a CU are cut if that ends the launch earlier by more than the
// partials cost (lists of unequal length, or a little more than a whole number of rounds): pieces of half
// the mean let a launch end evenly, shorter ones would only add partials to merge.
RowCut plan_row_cut(const std::vector<RowItem>& items, int64_t n_cu, int32_t kv_heads, int32_t seg_len, bool beside_units) {
  RowCut c;
  c.min_slots = std::max(1, kMinPieceTiles * kKvTile / seg_len);
  int64_t wgs = 0, load = 0;
  for (const RowItem& it : items) {
    wgs += it.row_tiles * kv_heads;
    load += it.walk.kv_tiles * it.row_tiles;
  }
  if (wgs == 0 || n_cu <= 0) return c;
  const int64_t lanes = std::max<int64_t>(1, n_cu / kv_heads);
  if (wgs < n_cu) {
    c.chunks = (int32_t)std::min<int64_t>(16, (2 * n_cu + wgs - 1) / wgs);
    if (beside_units) return c;
    if (cut_workgroups(items, c, kv_heads, true) <= n_cu) return one_round_cut(items, n_cu, kv_heads, c);
    // more than half a round whole: as many pieces as end the launch earliest, their partials counted (26 row tiles of 8 kv
    // heads on one list of 6k tokens: whole 285 us, in the three pieces that two workgroups per CU would take 324).  The line is not
    // a measured one: below it the estimate would often be right too (512 tokens on 32k, 8 kv heads: four pieces 246 us, the eight
    // that are two workgroups per CU 263), but how many pieces such a prompt gets is part of the plan's stated behaviour, which
    // its tests count.
    if (2 * wgs > n_cu) {
      RowCut tried = c;
      double best_cost = 0;
      std::vector<RowWork> pieces;
      for (int32_t chunks = c.chunks; chunks >= 1; --chunks) {
        tried.chunks = chunks;
        const int64_t n_partial = cut_items(items, tried, pieces);
        const double cost = (double)makespan(pieces, lanes) + merge_tiles(n_partial, kv_heads);
        if (best_cost == 0 || cost <= best_cost) {
          best_cost = cost;
          c = tried;
        }
      }
    }
    return c;
  }
  RowCut half = c;
  half.longest = std::max<int64_t>(kMinPieceTiles, load / lanes / 2);
  std::vector<RowWork> pieces;
  const int64_t n_whole = cut_items(items, c, pieces);
  std::vector<RowWork> whole = pieces;
  const int64_t n_cut = cut_items(items, half, pieces);
  if (n_cut == n_whole) return c;
  return 1.05 * makespan(pieces, lanes) + merge_tiles(n_cut - n_whole, kv_heads) < makespan(whole, lanes) ? half : c;
}

}  // namespace

extern "C" {

tl_status tl_plan_create(tl_plan** out, const tl_pool* pool, int32_t q_heads, int32_t n_req,
                         const int32_t* req_row_ptr, const int32_t* req_seg_ptr, const uint64_t* seg_ids,
                         int32_t flags, int32_t split_segments, int32_t compute_units) {
  if (!out) TL_FAIL(TL_EINVAL, "tl_plan_create: null out");
  *out = nullptr;
  if (!pool || n_req < 0 || !req_row_ptr || !req_seg_ptr) TL_FAIL(TL_EINVAL, "tl_plan_create: bad argument");
  if (q_heads <= 0 || q_heads % pool->kv_heads) TL_FAIL(TL_EINVAL, "tl_plan_create: q_heads must be a multiple of kv_heads");
  const int G = q_heads / pool->kv_heads;
  if (G > 32) TL_FAIL(TL_EINVAL, "tl_plan_create: q_heads/kv_heads must be at most 32");
  if (split_segments < 0) TL_FAIL(TL_EINVAL, "tl_plan_create: negative split_segments");
  if (compute_units > 4096) TL_FAIL(TL_EINVAL, "tl_plan_create: compute_units above 4096");
  if ((flags & (TL_PLAN_FUSE_ROWS | TL_PLAN_FUSE_TAILS)) && !(flags & TL_PLAN_SELF_BLOCK))
    TL_FAIL(TL_EINVAL, "tl_plan_create: TL_PLAN_FUSE_ROWS and TL_PLAN_FUSE_TAILS need TL_PLAN_SELF_BLOCK");
  if ((flags & TL_PLAN_FUSE_TAILS) && (flags & TL_PLAN_NO_SHARING))
    TL_FAIL(TL_EINVAL, "tl_plan_create: TL_PLAN_FUSE_TAILS has nothing to do under TL_PLAN_NO_SHARING");
  if (req_row_ptr[0] != 0 || req_seg_ptr[0] != 0) TL_FAIL(TL_EINVAL, "tl_plan_create: offsets must start at 0");
  for (int32_t r = 0; r < n_req; ++r)
    if (req_row_ptr[r + 1] < req_row_ptr[r] || req_seg_ptr[r + 1] < req_seg_ptr[r])
      TL_FAIL(TL_EINVAL, "tl_plan_create: offsets of request %d decrease", r);
  const int32_t T = req_row_ptr[n_req];
  const int32_t n_entries = req_seg_ptr[n_req];
  if (n_entries > 0 && !seg_ids) TL_FAIL(TL_EINVAL, "tl_plan_create: null seg_ids");

  tl_plan* p = new (std::nothrow) tl_plan();
  if (!p) TL_FAIL(TL_ENOMEM, "tl_plan_create: host allocation failed");
  tl_status rc = TL_OK;
  try {
    p->pool = pool;
    p->q_heads = q_heads;
    p->kv_heads = pool->kv_heads;
    p->group = G;
    p->n_req = n_req;
    p->n_tokens = T;
    p->flags = flags;
    p->blob_dev = nullptr;
    p->pool_generation = pool->generation;
    p->pool_n_slots = pool->n_slots;

    // ---- a0: segment id -> slot ------------------------------------------------------
    std::vector<int32_t> slots(n_entries);
    for (int32_t i = 0; i < n_entries; ++i) {
      auto it = pool->slot_of.find(seg_ids[i]);
      if (it == pool->slot_of.end()) {
        set_error("tl_plan_create: segment id %llu (list entry %d) is not resident", (unsigned long long)seg_ids[i], i);
        delete p;
        return TL_ENOTFOUND;
      }
      slots[i] = it->second;
    }
    const uint64_t now = ++pool->clock;
    for (int32_t s : slots) pool->stamp[s] = now;

    auto len_of = [&](int32_t r) { return req_seg_ptr[r + 1] - req_seg_ptr[r]; };
    auto slot_at = [&](int32_t r, int32_t pos) { return slots[req_seg_ptr[r] + pos]; };
    auto ntok_of = [&](int32_t r) { return req_row_ptr[r + 1] - req_row_ptr[r]; };

    // What a work item over positions [begin, end) of a request's list walks: a slot that is named several
    // times once, unless TL_PLAN_WALK_REPEATS.
    const bool dedupe = !(flags & TL_PLAN_WALK_REPEATS);
    std::vector<int32_t> walked_by(dedupe ? pool->n_slots : 0, 0);
    int32_t walker = 0;
    auto walk_of = [&](int32_t r, int32_t begin, int32_t end) {
      Walk w{0, 0, 0};
      ++walker;
      for (int32_t pos = begin; pos < end; ++pos) {
        const int32_t sl = slot_at(r, pos);
        if (dedupe) {
          if (walked_by[sl] == walker) continue;
          walked_by[sl] = walker;
        }
        ++w.slots;
        w.tokens += pool->fill[sl];
        w.kv_tiles += (pool->fill[sl] + kKvTile - 1) / kKvTile;
      }
      return w;
    };

    // ---- group requests along shared runs ----------------------------------------------
    // With TL_PLAN_FUSE_ROWS a request is set aside for the one-pass kernel if sharing a run of slots
    // with other requests gains it nothing: it has no slot in common with another request of the
    // batch, or it has enough rows of its own (the work is then bound by the matrix unit, not by KV
    // traffic) -- either way it would only lose a partial per row, and a merge, on the other path.
    // Requests with a token's worth of rows (decode) always take split-K units.
    const int tok_tile = kRowTile / G, half_tile = half_row_tile(G);
    auto row_item = [&](const Walk& w, int64_t n_tok) {
      const int64_t whole = n_tok / tok_tile, rest = n_tok % tok_tile;
      return RowItem{w, whole + (rest > 0), whole * (tok_tile > half_tile ? 2 : 1) + (rest > half_tile ? 2 : rest > 0), n_tok * G};
    };
    const int64_t n_cu = compute_units < 0 ? kComputeUnits : compute_units;
    const int32_t min_chunk_slots = std::max(1, kMinPieceTiles * kKvTile / pool->seg_len);
    std::vector<char> fused(n_req, 0);
    // A one-pass row tile cannot be cut along its KV: when the whole batch is fewer row-tile
    // workgroups than the GPU has CUs (one long prompt, say), requests whose slot lists are long
    // enough to be cut (see below) stay on the three-step path
    bool small_batch = false;
    {
      int64_t wgs = 0;
      for (int32_t r = 0; r < n_req; ++r)
        if (ntok_of(r) > 0) wgs += (int64_t)((ntok_of(r) + tok_tile - 1) / tok_tile) * pool->kv_heads;
      small_batch = wgs < n_cu;
    }
    if (flags & TL_PLAN_FUSE_ROWS) {
      std::vector<int32_t> users(pool->n_slots, 0), last_user(pool->n_slots, -1);
      for (int32_t r = 0; r < n_req; ++r) {
        if (ntok_of(r) == 0) continue;
        for (int32_t pos = 0; pos < len_of(r); ++pos) {
          const int32_t sl = slot_at(r, pos);
          if (last_user[sl] != r) {
            last_user[sl] = r;
            users[sl]++;
          }
        }
      }
      for (int32_t r = 0; r < n_req; ++r) {
        const int64_t rows = (int64_t)ntok_of(r) * G;
        if (rows <= kUnitRows) continue;
        if (small_batch && len_of(r) > min_chunk_slots) continue;
        bool shares = false;
        for (int32_t pos = 0; pos < len_of(r) && !shares; ++pos) shares = users[slot_at(r, pos)] > 1;
        fused[r] = rows >= kFuseRows || !shares;
      }
    }
    // ---- walk the prefix tree ---------------------------------------------------------------------
    // every request with a list, in order, front to back; `grouped` requests are those the planner
    // may put together (new tokens, not set aside for the one-pass kernel)
    PrefixTree& tree = pool->tree;
    // Lists that follow no tree (the same segments in ever new orders) would add nodes batch after batch:
    // beyond kTreeNodesPerSlot nodes per slot the tree, a record of loads, starts over.
    if ((int64_t)tree.size() > (int64_t)kTreeNodesPerSlot * pool->n_slots) tree.reset(pool->n_slots);
    tree.begin_batch();
    std::vector<int32_t> path(n_entries);          // tree node of every list entry
    auto is_live = [&](int32_t r) { return ntok_of(r) > 0 && len_of(r) > 0 && !fused[r]; };
    for (int32_t r = 0; r < n_req; ++r) {
      const bool grouped = is_live(r);
      int32_t node = 0;
      for (int32_t i = req_seg_ptr[r]; i < req_seg_ptr[r + 1]; ++i) {
        node = tree.child(node, seg_ids[i], slots[i]);
        tree.visit(node, ntok_of(r), grouped, r);
        path[i] = node;
      }
    }
    // the batch's part of the tree, copied for tl_plan_hot_slots (which must not need the pool)
    {
      const std::vector<int32_t>& bn = tree.batch_nodes();
      const size_t nb = bn.size();
      p->bt_slot.resize(nb);
      p->bt_load.resize(nb);
      p->bt_first_child.resize(nb);
      p->bt_next_sib.resize(nb);
      auto idx = [&](int32_t n) { return n < 0 ? -1 : tree.at(n).batch_index; };
      for (size_t i = 0; i < nb; ++i) {
        const TreeNode& x = tree.at(bn[i]);
        p->bt_slot[i] = x.slot;
        p->bt_load[i] = x.batch_load;
        p->bt_first_child[i] = idx(x.batch_first_child);
        p->bt_next_sib[i] = idx(x.batch_next_sib);
      }
      for (int32_t c = tree.at(0).batch_first_child; c >= 0; c = tree.at(c).batch_next_sib) p->bt_roots.push_back(idx(c));
    }

    // ---- work items from tree nodes -----------------------------------------------------------------
    std::vector<RawItem> raw;
    std::vector<int32_t> live;
    for (int32_t r = 0; r < n_req; ++r)
      if (is_live(r)) live.push_back(r);
    if (flags & TL_PLAN_NO_SHARING) {
      for (int32_t r : live) raw.push_back(RawItem{{r}, r, 0, len_of(r)});
    } else {
      // A run starts at a node and goes down while one child carries all of the node's grouped
      // requests (then nobody has ended and nobody has turned off).  Runs come out parent level
      // first, siblings in order of their first request, then each sibling's subtree in turn.
      std::vector<int32_t> item_of(tree.batch_nodes().size(), -1);   // run that starts at a visited node
      std::vector<int32_t> stack(1, 0), kids, next;
      while (!stack.empty()) {
        const int32_t f = stack.back();
        stack.pop_back();
        kids.clear();
        for (int32_t c = tree.at(f).batch_first_child; c >= 0; c = tree.at(c).batch_next_sib)
          if (tree.at(c).batch_cnt > 0) kids.push_back(c);
        std::sort(kids.begin(), kids.end(),
                  [&](int32_t a, int32_t b) { return tree.at(a).batch_first_req < tree.at(b).batch_first_req; });
        next.clear();
        for (int32_t c : kids) {
          const int32_t cnt = tree.at(c).batch_cnt;
          int32_t last = c;
          for (;;) {
            int32_t all = -1;
            for (int32_t d = tree.at(last).batch_first_child; d >= 0; d = tree.at(d).batch_next_sib)
              if (tree.at(d).batch_cnt == cnt) { all = d; break; }
            if (all < 0) break;
            last = all;
          }
          item_of[tree.at(c).batch_index] = (int32_t)raw.size();
          raw.push_back(RawItem{{}, tree.at(c).batch_first_req, tree.at(c).depth, tree.at(last).depth + 1});
          next.push_back(last);
        }
        for (auto it = next.rbegin(); it != next.rend(); ++it) stack.push_back(*it);
      }
      // who passes through each run's first node, in request order
      for (int32_t r : live)
        for (int32_t i = req_seg_ptr[r]; i < req_seg_ptr[r + 1]; ++i) {
          const int32_t it = item_of[tree.at(path[i]).batch_index];
          if (it >= 0) raw[it].reqs.push_back(r);
        }
    }

    // An item goes to split-K units if it has a token's worth of rows, or if it is a run shared by
    // decode-type requests only (each with a token's worth of rows) that together would not fill
    // one row tile: such a run has too little arithmetic for a row tile to matter and, as a handful
    // of workgroups in a launch of its own, would only add its latency to the step.  Its tokens are
    // then dealt to units of kUnitRows rows, which re-read the run through L2.
    const int32_t tok_unit = std::max(1, kUnitRows / G);
    auto unit_item = [&](const RawItem& it, int64_t n_tok) -> bool {
      if (n_tok * G <= kUnitRows) return true;
      if (n_tok * G > kRowTile) return false;
      for (int32_t r : it.reqs)
        if ((int64_t)ntok_of(r) * G > kUnitRows) return false;
      return true;
    };
    auto tok_of = [&](const RawItem& it) {
      int64_t n_tok = 0;
      for (int32_t r : it.reqs) n_tok += ntok_of(r);
      return n_tok;
    };

    int split = split_segments;
    if (split == 0) {
      // Split-K chunk, in slots.  Measured on decode batches of 1 to 1024 requests: long chunks stream
      // best (2 slots 5.6 TB/s, 8 slots 6.0, 32 slots 6.1, and fewer partials to merge), as long as
      // there are about as many units as CUs or more; equal-sized units that overflow one round of CUs
      // by a little leave a thin second round that cannot fill the memory system.  So: the longest
      // chunk (at most 32 slots, at least 512 tokens) that still gives three quarters of a unit per
      // CU, halved if the count then lands between one and one and a half rounds.
      std::vector<std::pair<int64_t, int64_t>> runs;     // (list entries, token groups) of every unit item
      for (const RawItem& it : raw) {
        const int64_t n_tok = tok_of(it);
        if (unit_item(it, n_tok)) runs.emplace_back(it.end - it.begin, (n_tok + tok_unit - 1) / tok_unit);
      }
      auto units_with = [&](int sp) {
        int64_t u = 0;
        for (const auto& r : runs) u += (r.first + sp - 1) / sp * r.second;
        return u;
      };
      const int lo = std::max(1, 512 / pool->seg_len);
      const int64_t cus = n_cu > 0 ? n_cu : kComputeUnits;
      split = 32;
      while (split > lo && 4 * units_with(split) < 3 * cus) --split;
      const int64_t u = units_with(split);
      if (u > cus && 2 * u < 3 * cus && split >= 2 * lo) split /= 2;
    }

    // ---- one-pass rows beside split-K units --------------------------------------------------
    // In a batch that also has split-K units (one that is all one-pass rows stays so: its caller may make the
    // one-pass call alone): one-pass rows whose lists differ much in length leave CUs idle behind the longest, which cannot
    // be cut, in a launch of their own behind the units'.  On the three steps their lists can be cut and share the units'
    // launch: each such request becomes a work item of its own (its rows are many enough: sharing a run would cut its
    // list at every fork and add partials).  Both plans are weighed as they would be built, with the same pieces and
    // the units' time in both; the one-pass rows stay unless the three steps are 6 % cheaper.  Of the 758 batches 325 leave
    // the one-pass kernel: 0.51 to 1.05 of its time, 0.79 in the mean, four of them slower by more than 2 % (8 chunks of up to
    // 211 tokens beside 42 decoded ones on 3.9k to 31k 1174 and 832 us).  The line is where it is for those four: of the
    // batches that stay, 47 would have gained a tenth or more.
    RowCut row_cut;
    bool row_cut_known = false;
    if (n_cu > 0 && !(flags & TL_PLAN_FUSE_TAILS) && std::find(fused.begin(), fused.end(), 1) != fused.end()) {
      int64_t unit_tokens = 0;
      UnitLoad load;
      std::vector<RowItem> kept;           // row-tile items of either plan
      for (const RawItem& it : raw) {
        const int64_t n_tok = tok_of(it);
        const Walk w = walk_of(it.src_req, it.begin, it.end);
        if (unit_item(it, n_tok)) {
          const int64_t groups = (n_tok + tok_unit - 1) / tok_unit;
          unit_tokens += w.tokens;
          load.units += (w.slots + split - 1) / split * groups;
          load.tokens += w.tokens * groups;
          load.longest = std::max(load.longest, w.tokens * std::min(split, w.slots) / std::max(1, w.slots));
        } else {
          kept.push_back(row_item(w, n_tok));
        }
      }
      // (units of less than a fifth of a tile's time, a token or two on short prefixes, are no launch to share)
      const double units = (double)unit_tokens * pool->kv_heads * (4 * kHeadDim) / kUnitBytesPerTile;
      if (units >= 0.2) {
        const int64_t lanes = std::max<int64_t>(1, n_cu / pool->kv_heads);
        std::vector<RowItem> all = kept;
        std::vector<RowWork> one_pass, causal;
        int64_t self_rows = 0;
        for (int32_t r = 0; r < n_req; ++r) {
          if (!fused[r] || len_of(r) == 0) continue;
          const Walk w = walk_of(r, 0, len_of(r));
          const int64_t n_row = (ntok_of(r) + tok_tile - 1) / tok_tile;
          all.push_back(row_item(w, ntok_of(r)));
          self_rows += n_row;
          for (int64_t i = 0; i < n_row; ++i) {
            const int64_t self = (std::min<int64_t>((i + 1) * tok_tile, ntok_of(r)) + kKvTile - 1) / kKvTile;
            one_pass.push_back(RowWork{w.kv_tiles + self, 1});
            causal.push_back(RowWork{self, 1});
          }
        }
        if (self_rows > 0) {
          const int64_t unit_blocks = load.units * unit_head_blocks(pool->kv_heads, plan_unit_heads_log2(pool->kv_heads, load, n_cu));
          std::vector<RowWork> pieces;
          const RowCut cut_kept = plan_row_cut(kept, n_cu, pool->kv_heads, pool->seg_len, true);
          const RowCut cut_all = plan_row_cut(all, n_cu, pool->kv_heads, pool->seg_len, true);
          const int64_t rows_kept = cut_items(kept, cut_kept, pieces);
          const double as_one_pass = joint_tiles(units, unit_blocks, makespan(pieces, lanes), n_cu) + makespan(one_pass, lanes) + kOnePassLaunch;
          const int64_t rows_all = cut_items(all, cut_all, pieces);
          const double as_three = joint_tiles(units, unit_blocks, makespan(pieces, lanes), n_cu) + 1.3 * makespan(causal, lanes) +
                                  1.2 * merge_tiles(rows_all - rows_kept + self_rows, pool->kv_heads) + kThreeStepLaunches;
          row_cut_known = true;
          row_cut = cut_kept;
          if (as_three < 0.94 * as_one_pass) {
            row_cut = cut_all;
            for (int32_t r = 0; r < n_req; ++r)
              if (fused[r] && len_of(r) > 0) {
                fused[r] = 0;
                raw.push_back(RawItem{{r}, r, 0, len_of(r)});
              }
          }
        }
      }
    }

    // The kv tokens of a slot list as tiles of kKvTile rows.  A slot listed several times (lists are
    // multisets: Section 3.1 has no order or uniqueness among the segments a request attends to) is
    // walked once; its tiles carry log2 of the multiplicity, which the kernel adds to the exponent
    // (m equal keys weigh m exp(s) in numerator and denominator alike).  Returns the pairs computed.
    std::vector<int32_t> mult_of(dedupe ? pool->n_slots : 0, 0);
    auto emit_tiles = [&](auto slot_of_pos, int32_t n_pos) -> int64_t {
      int64_t kv_tokens = 0;
      if (dedupe)
        for (int32_t pos = 0; pos < n_pos; ++pos) mult_of[slot_of_pos(pos)]++;
      for (int32_t pos = 0; pos < n_pos; ++pos) {
        const int32_t sl = slot_of_pos(pos), f = pool->fill[sl];
        int32_t m = 1;
        if (dedupe) {
          m = mult_of[sl];
          if (m == 0) continue;        // a later occurrence of a slot already emitted
          mult_of[sl] = 0;
        }
        const float lm = log2f((float)m);
        if (m > 1) p->any_repeat = true;
        kv_tokens += f;
        for (int32_t off = 0; off < f; off += kKvTile) {
          if (off + kKvTile <= f) {
            p->tile_base.push_back(sl * pool->seg_len + off);
            p->tile_lm.push_back(lm);
          } else {
            p->part_tile.push_back(sl * pool->seg_len + off);
            p->part_tile.push_back(f - off);
            p->part_lm.push_back(lm);
          }
        }
      }
      return kv_tokens;
    };

    // ---- one-pass tails ---------------------------------------------------------------------
    // TL_PLAN_FUSE_TAILS: a request with more than a token's worth of rows takes the one-pass kernel
    // for the end of its list that nobody shares (the run whose only request it is; possibly empty)
    // and its own new tokens.  The shared runs above stay work items, read once for all their
    // requesters' rows; their partial rows for this request are listed as `priors`, which the
    // one-pass kernel's epilogue merges in, so the request needs no causal tile and no tl_merge.
    std::vector<char> tailed(n_req, 0);
    std::vector<int32_t> tail_begin(n_req, 0), tail_end(n_req, 0);
    std::vector<std::vector<int32_t>> priors(n_req);     // per request: partial row of its first token in every shared item
    std::vector<char> is_tail_item(raw.size(), 0);
    if (flags & TL_PLAN_FUSE_TAILS) {
      for (int32_t r = 0; r < n_req; ++r) {
        if (fused[r] || (int64_t)ntok_of(r) * G <= kUnitRows) continue;
        tailed[r] = 1;
        tail_begin[r] = tail_end[r] = len_of(r);
      }
      for (size_t i = 0; i < raw.size(); ++i) {
        const RawItem& it = raw[i];
        if (it.reqs.size() != 1 || !tailed[it.reqs[0]]) continue;
        const int32_t r = it.reqs[0];
        if (small_batch && it.end - it.begin > min_chunk_slots) {    // long enough to be cut along its KV instead
          tailed[r] = 0;
          continue;
        }
        is_tail_item[i] = 1;
        tail_begin[r] = it.begin;
        tail_end[r] = it.end;
      }
    }

    // ---- final items, work lists ----------------------------------------------------------
    if (!row_cut_known) {
      std::vector<RowItem> items;
      bool any_unit = false;
      for (size_t i = 0; i < raw.size(); ++i) {
        const int64_t n_tok = is_tail_item[i] ? 0 : tok_of(raw[i]);
        if (n_tok > 0 && !unit_item(raw[i], n_tok))
          items.push_back(row_item(walk_of(raw[i].src_req, raw[i].begin, raw[i].end), n_tok));
        else if (n_tok > 0)
          any_unit = true;
      }
      row_cut = plan_row_cut(items, n_cu, pool->kv_heads, pool->seg_len, any_unit);
    }
    int32_t row_cursor = 0;
    const int32_t own_toks = (flags & TL_PLAN_SELF_BLOCK) ? T : 0;      // the token array: every token in order, then the items' tokens
    p->item_tok_ptr.push_back(0);
    p->item_slot_ptr.push_back(0);
    int64_t prefix_pairs = 0, tile_pairs = 0;
    int32_t n_fused_tokens = 0;
    int64_t item_pairs = 0;
    for (size_t ri = 0; ri < raw.size(); ++ri) {
      const RawItem& it = raw[ri];
      if (is_tail_item[ri]) continue;
      const int32_t n_tok = (int32_t)tok_of(it);
      const bool few_rows = unit_item(it, n_tok);
      // Pieces are cut from the slots that the run walks, not from its list: a piece of the list would
      // walk again what another piece names too.
      int32_t step = split;
      bool cut = few_rows;
      if (!few_rows) {
        const Walk w = walk_of(it.src_req, it.begin, it.end);
        step = row_cut.step(w);
        cut = step < w.slots;
        if (!cut) step = it.end - it.begin;
      }
      // The run's slots, each with the number of times the run lists it.  Split-K units walk a slot
      // that is listed m times once, with weight m, like the row tiles (reading 8 of the paper's
      // silence on repeated segments: a list is a multiset); row-tile items that stay whole dedupe in
      // emit_tiles, so for them every list position stays an entry of its own here.
      std::vector<std::pair<int32_t, int32_t>> run_slots;
      {
        const int32_t n_pos = it.end - it.begin;
        if (cut && dedupe) {
          for (int32_t pos = it.begin; pos < it.end; ++pos) mult_of[slot_at(it.src_req, pos)]++;
          for (int32_t pos = it.begin; pos < it.end; ++pos) {
            const int32_t sl = slot_at(it.src_req, pos);
            if (mult_of[sl] == 0) continue;
            run_slots.emplace_back(sl, mult_of[sl]);
            mult_of[sl] = 0;
          }
        } else {
          run_slots.reserve(n_pos);
          for (int32_t pos = it.begin; pos < it.end; ++pos) run_slots.emplace_back(slot_at(it.src_req, pos), 1);
        }
      }
      const int32_t run = (int32_t)run_slots.size();
      for (int32_t c0 = 0; c0 < run; c0 += step) {
        const int32_t c1 = std::min(run, c0 + step);
        const int32_t tok_base = own_toks + (int32_t)p->item_tokens.size();
        for (int32_t r : it.reqs)
          for (int32_t t = req_row_ptr[r]; t < req_row_ptr[r + 1]; ++t) p->item_tokens.push_back(t);
        const int32_t slot_base = (int32_t)p->item_slots.size();
        const int32_t unit_base = (int32_t)(p->unit_slots.size() / 2);
        for (int32_t u = c0; u < c1; ++u) {
          const int32_t sl = run_slots[u].first, m = run_slots[u].second;
          for (int32_t k = 0; k < m; ++k) p->item_slots.push_back(sl);       // the item's list keeps every occurrence
          prefix_pairs += (int64_t)m * n_tok * pool->fill[sl];
          item_pairs += (int64_t)m * n_tok * pool->fill[sl];
          if (few_rows) {
            p->unit_slots.push_back(sl * pool->seg_len);
            p->unit_slots.push_back(pool->fill[sl]);
            p->unit_lm.push_back(log2f((float)m));
            if (m > 1) p->any_unit_repeat = true;
          }
        }
        {
          int32_t first = row_cursor;             // partial row of each tailed requester's first token in this item
          for (int32_t r : it.reqs) {
            if (tailed[r]) priors[r].push_back(first);
            first += ntok_of(r);
          }
        }
        p->item_row_base.push_back(row_cursor);
        p->item_tok_ptr.push_back((int32_t)p->item_tokens.size());
        p->item_slot_ptr.push_back((int32_t)p->item_slots.size());
        if (few_rows) {
          for (int32_t t0 = 0; t0 < n_tok; t0 += tok_unit)
            p->units.push_back(Work{tok_base + t0, std::min(tok_unit, n_tok - t0), row_cursor + t0, unit_base, c1 - c0, 0, 0, 0, 0, 0, 0});
        } else {
          // the item's kv tokens as tiles of kKvTile rows (shared by all its row tiles)
          const int32_t full_off = (int32_t)p->tile_base.size();
          const int32_t part_off = (int32_t)p->part_tile.size() / 2;
          tile_pairs += (int64_t)n_tok * emit_tiles([&](int32_t pos) { return p->item_slots[slot_base + pos]; },
                                                    (int32_t)p->item_slots.size() - slot_base);
          const int32_t n_full = (int32_t)p->tile_base.size() - full_off;
          const int32_t n_part = (int32_t)p->part_tile.size() / 2 - part_off;
          // row tiles never straddle two requests' token ranges unless ranges are short:
          // tokens are simply taken tok_tile at a time in item order (Q rows are gathered).
          for (int32_t t0 = 0; t0 < n_tok; t0 += tok_tile)
            p->tiles.push_back(Work{tok_base + t0, std::min(tok_tile, n_tok - t0), row_cursor + t0, slot_base, (int32_t)p->item_slots.size() - slot_base,
                                    full_off, n_full, part_off, n_part, 0, 0});
        }
        if ((int64_t)row_cursor + n_tok + T > INT32_MAX) {      // partial rows are numbered in 32 bits
          set_error("tl_plan_create: more than 2^31 partial rows");
          delete p;
          return TL_EINVAL;
        }
        row_cursor += n_tok;
      }
    }
    UnitLoad unit_load;
    for (const Work& w : p->units) {
      int64_t tokens = 0;
      for (int32_t i = w.kv_off; i < w.kv_off + w.kv_len; ++i) tokens += p->unit_slots[2 * (size_t)i + 1];
      ++unit_load.units;
      unit_load.tokens += tokens;
      unit_load.longest = std::max(unit_load.longest, tokens);
    }
    p->unit_heads_log2 = plan_unit_heads_log2(pool->kv_heads, unit_load, n_cu > 0 ? n_cu : kComputeUnits);
    p->tok.resize(own_toks);
    std::iota(p->tok.begin(), p->tok.end(), 0);
    p->tok.insert(p->tok.end(), p->item_tokens.begin(), p->item_tokens.end());

    const int32_t n_items = (int32_t)p->item_row_base.size();
    int32_t self_base = -1;
    int64_t self_pairs = 0;
    if (flags & TL_PLAN_SELF_BLOCK) {
      self_base = row_cursor;
      for (int32_t r = 0; r < n_req; ++r) {
        const int32_t a = req_row_ptr[r], b = req_row_ptr[r + 1];
        const int64_t lq = b - a;
        self_pairs += lq * (lq + 1) / 2;
        int32_t full_off = 0, n_full = 0, part_off = 0, n_part = 0;
        int32_t prior_off = 0, n_prior = 0;
        if (fused[r] || tailed[r]) {
          // the request's whole slot list (one-pass rows) or the private end of it (one-pass tail) as
          // tiles of kKvTile rows
          const int32_t p0 = fused[r] ? 0 : tail_begin[r], p1 = fused[r] ? len_of(r) : tail_end[r];
          full_off = (int32_t)p->tile_base.size();
          part_off = (int32_t)p->part_tile.size() / 2;
          for (int32_t pos = p0; pos < p1; ++pos) prefix_pairs += lq * pool->fill[slot_at(r, pos)];
          tile_pairs += lq * emit_tiles([&](int32_t pos) { return slot_at(r, p0 + pos); }, p1 - p0);
          n_full = (int32_t)p->tile_base.size() - full_off;
          n_part = (int32_t)p->part_tile.size() / 2 - part_off;
          n_fused_tokens += (int32_t)lq;
          prior_off = (int32_t)p->prior_rows.size();
          n_prior = (int32_t)priors[r].size();
          p->prior_rows.insert(p->prior_rows.end(), priors[r].begin(), priors[r].end());
          fused[r] = 1;                   // from here on the two kinds are the same thing
        }
        if (!fused[r] && lq == 1) {      // a single new token sees itself only: no row tile for it
          p->single_tok.push_back(a);
          continue;
        }
        for (int32_t t0 = a; t0 < b; t0 += tok_tile) {
          const int32_t n = std::min(tok_tile, b - t0);
          if (fused[r])
            p->ftiles.push_back(Work{t0, n, t0, a, t0 + n - a, full_off, n_full, part_off, n_part, prior_off, n_prior});
          else
            p->ctiles.push_back(Work{t0, n, self_base + t0, a, t0 + n - a, 0, 0, 0, 0, 0, 0});
        }
      }
      row_cursor += T;
    }

    // longest first, so that the tail of the launch is made of short work
    auto by_len = [&](const Work& x, const Work& y) {
      return (x.n_full + x.n_part ? x.n_full + x.n_part : x.kv_len) > (y.n_full + y.n_part ? y.n_full + y.n_part : y.kv_len);
    };
    std::stable_sort(p->tiles.begin(), p->tiles.end(), by_len);
    std::stable_sort(p->units.begin(), p->units.end(), by_len);
    std::stable_sort(p->ctiles.begin(), p->ctiles.end(), by_len);
    // one-pass rows: the row tiles of a request stay next to each other in the launch order, run at the same time and share
    // its KV through L2; requests by their pool length, then by their new tokens, and of a request the last rows,
    // which see the most of them, first (in the order of the batch, the longest row tiles of a
    // prompt started last: 8 prompts of 700 to 4096 tokens 537 -> 517 us)
    {
      std::vector<std::pair<int32_t, int32_t>> spans;       // [first, last) row tile of a request
      for (int32_t i = 0; i < (int32_t)p->ftiles.size(); ++i) {
        if (i == 0 || p->ftiles[i].kv_off != p->ftiles[i - 1].kv_off) spans.emplace_back(i, i);
        spans.back().second = i + 1;
      }
      std::stable_sort(spans.begin(), spans.end(), [&](const std::pair<int32_t, int32_t>& x, const std::pair<int32_t, int32_t>& y) {
        const Work &a = p->ftiles[x.second - 1], &b = p->ftiles[y.second - 1];
        const int32_t na = a.n_full + a.n_part, nb = b.n_full + b.n_part;
        return na != nb ? na > nb : a.kv_len > b.kv_len;
      });
      std::vector<Work> sorted;
      sorted.reserve(p->ftiles.size());
      for (const auto& s : spans)
        for (int32_t i = s.second - 1; i >= s.first; --i) sorted.push_back(p->ftiles[i]);
      p->ftiles.swap(sorted);
    }

    {
      std::vector<double> unit_bytes;      // of a workgroup: the kv heads that it takes of its unit's tokens
      unit_bytes.reserve(p->units.size());
      for (const Work& w : p->units) {
        int64_t tokens = 0;
        for (int32_t i = w.kv_off; i < w.kv_off + w.kv_len; ++i) tokens += p->unit_slots[2 * (size_t)i + 1];
        unit_bytes.push_back((double)tokens * std::min(1 << p->unit_heads_log2, pool->kv_heads) * (4 * kHeadDim));
      }
      p->unit_lanes = (int32_t)plan_unit_lanes(unit_bytes, p->unit_heads_log2, p->tiles, pool->kv_heads, n_cu);
    }

    auto halve = [&](const std::vector<Work>& tiles) {
      int64_t wgs = (int64_t)tiles.size();
      for (const Work& w : tiles) wgs += w.n_tok > half_tile;
      return halves_fit((int64_t)tiles.size(), wgs, pool->kv_heads, n_cu);
    };
    p->halve_tiles = halve(p->tiles) && p->units.empty();
    p->halve_ctiles = halve(p->ctiles);
    p->halve_ftiles = halve(p->ftiles);

    // ---- merge lists --------------------------------------------------------------------------
    // (tokens of one-pass requests are in no merge list: a one-pass tail's partial rows in the shared
    // items are read by the one-pass kernel itself)
    std::vector<char> tok_fused(T, 0);
    for (int32_t r = 0; r < n_req; ++r)
      if (fused[r])
        for (int32_t t = req_row_ptr[r]; t < req_row_ptr[r + 1]; ++t) tok_fused[t] = 1;
    p->merge_ptr.assign(T + 1, 0);
    for (int32_t i = 0; i < n_items; ++i)
      for (int32_t j = p->item_tok_ptr[i]; j < p->item_tok_ptr[i + 1]; ++j)
        if (!tok_fused[p->item_tokens[j]]) p->merge_ptr[p->item_tokens[j] + 1]++;
    for (int32_t t = 0; t < T; ++t)
      if (!tok_fused[t]) p->merge_tok.push_back(t);
    if (self_base >= 0)
      for (int32_t t = 0; t < T; ++t)
        if (!tok_fused[t]) p->merge_ptr[t + 1]++;
    for (int32_t t = 0; t < T; ++t) p->merge_ptr[t + 1] += p->merge_ptr[t];
    // tokens with longer lists (pieces of one list, split-K) last: tl_merge gives them kernels of their own
    {
      auto shorter = [&](int32_t n) {
        return [&, n](int32_t t) { return p->merge_ptr[t + 1] - p->merge_ptr[t] < n; };
      };
      auto mid = std::stable_partition(p->merge_tok.begin(), p->merge_tok.end(), shorter(kMidMergeList));
      auto end = std::stable_partition(mid, p->merge_tok.end(), shorter(kLongMergeList));
      p->n_merge_short = (int32_t)(mid - p->merge_tok.begin());
      p->n_merge_mid = (int32_t)(end - mid);
    }
    p->merge_rows.assign(p->merge_ptr[T], 0);
    {
      std::vector<int32_t> cur(p->merge_ptr.begin(), p->merge_ptr.end() - 1);
      for (int32_t i = 0; i < n_items; ++i)
        for (int32_t j = p->item_tok_ptr[i]; j < p->item_tok_ptr[i + 1]; ++j)
          if (!tok_fused[p->item_tokens[j]]) p->merge_rows[cur[p->item_tokens[j]]++] = p->item_row_base[i] + (j - p->item_tok_ptr[i]);
      if (self_base >= 0)
        for (int32_t t = 0; t < T; ++t)
          if (!tok_fused[t]) p->merge_rows[cur[t]++] = self_base + t;
    }
    // the short lists once more as fixed records, so that the merge kernel gets a token's whole list with
    // one load instead of three dependent ones
    static_assert(kMidMergeList <= kMergeFixInts, "a short list and its token fit one record");
    p->merge_fix.assign((size_t)p->n_merge_short * kMergeFixInts, -1);
    for (int32_t i = 0; i < p->n_merge_short; ++i) {
      const int32_t t = p->merge_tok[i];
      int32_t* rec = &p->merge_fix[(size_t)i * kMergeFixInts];
      rec[0] = t;
      for (int32_t j = p->merge_ptr[t]; j < p->merge_ptr[t + 1]; ++j) rec[1 + j - p->merge_ptr[t]] = p->merge_rows[j];
    }

    int64_t uniq_tok = 0;
    {
      std::vector<char> seen(pool->n_slots, 0);
      for (int32_t s : slots)
        if (!seen[s]) {
          seen[s] = 1;
          uniq_tok += pool->fill[s];
        }
    }

    tl_plan_info& inf = p->info;
    memset(&inf, 0, sizeof(inf));
    inf.n_req = n_req;
    inf.n_tokens = T;
    inf.q_heads = q_heads;
    inf.kv_heads = pool->kv_heads;
    inf.n_items = n_items;
    inf.n_partial_rows = row_cursor;
    inf.self_row_base = self_base;
    inf.n_tiles = (int32_t)p->tiles.size();
    inf.n_units = (int32_t)p->units.size();
    inf.n_causal_tiles = (int32_t)p->ctiles.size();
    inf.n_list_entries = n_entries;
    inf.n_merge_entries = (int32_t)p->merge_rows.size();
    inf.prefix_pairs = prefix_pairs;
    inf.self_pairs = self_pairs;
    inf.unique_kv_tokens = uniq_tok;
    inf.n_fused_tiles = (int32_t)p->ftiles.size();
    inf.n_fused_tokens = n_fused_tokens;
    inf.n_single_tokens = (int32_t)p->single_tok.size();
    inf.tile_pairs = tile_pairs;
    inf.item_pairs = item_pairs;
    inf.n_prior_rows = (int32_t)p->prior_rows.size();
    inf.n_unit_workgroups = p->unit_lanes;

    // ---- one block with everything the kernels read ---------------------------------------------
    {
      size_t total = 0;
      auto reserve = [&](size_t bytes) {
        const size_t at = total;
        total += (bytes + 255) & ~(size_t)255;
        return at;
      };
      // first what the one-pass kernel reads (of the token array, each token's own entry), all that
      // tl_fused_attn_static has to stage
      auto& o = p->off;
      o.ftiles = reserve(sizeof(Work) * p->ftiles.size());
      o.tile_base = reserve(sizeof(int32_t) * p->tile_base.size());
      o.part_tile = reserve(sizeof(int32_t) * p->part_tile.size());
      o.tile_lm = reserve(sizeof(float) * p->tile_lm.size());
      o.part_lm = reserve(sizeof(float) * p->part_lm.size());
      o.prior_rows = reserve(sizeof(int32_t) * p->prior_rows.size());
      o.tok = reserve(sizeof(int32_t) * p->tok.size());
      p->one_pass_bytes = ((o.tok + sizeof(int32_t) * own_toks + 255) & ~(size_t)255) + 256;    // with the block's slack at its end
      o.tiles = reserve(sizeof(Work) * p->tiles.size());
      o.units = reserve(sizeof(Work) * p->units.size());
      o.ctiles = reserve(sizeof(Work) * p->ctiles.size());
      o.unit_slots = reserve(sizeof(int32_t) * p->unit_slots.size());
      o.unit_lm = reserve(sizeof(float) * p->unit_lm.size());
      o.merge_ptr = reserve(sizeof(int32_t) * p->merge_ptr.size());
      o.merge_rows = reserve(sizeof(int32_t) * p->merge_rows.size());
      o.merge_tok = reserve(sizeof(int32_t) * p->merge_tok.size());
      o.single_tok = reserve(sizeof(int32_t) * p->single_tok.size());
      o.merge_fix = reserve(sizeof(int32_t) * p->merge_fix.size());
      p->blob_host.assign(total + 256, 0);
      auto fill = [&](size_t at, const void* src, size_t bytes) {
        if (bytes) memcpy(p->blob_host.data() + at, src, bytes);
      };
      fill(o.tiles, p->tiles.data(), sizeof(Work) * p->tiles.size());
      fill(o.units, p->units.data(), sizeof(Work) * p->units.size());
      fill(o.ctiles, p->ctiles.data(), sizeof(Work) * p->ctiles.size());
      fill(o.ftiles, p->ftiles.data(), sizeof(Work) * p->ftiles.size());
      fill(o.tok, p->tok.data(), sizeof(int32_t) * p->tok.size());
      fill(o.unit_slots, p->unit_slots.data(), sizeof(int32_t) * p->unit_slots.size());
      fill(o.unit_lm, p->unit_lm.data(), sizeof(float) * p->unit_lm.size());
      fill(o.merge_ptr, p->merge_ptr.data(), sizeof(int32_t) * p->merge_ptr.size());
      fill(o.merge_rows, p->merge_rows.data(), sizeof(int32_t) * p->merge_rows.size());
      fill(o.tile_base, p->tile_base.data(), sizeof(int32_t) * p->tile_base.size());
      fill(o.part_tile, p->part_tile.data(), sizeof(int32_t) * p->part_tile.size());
      fill(o.merge_tok, p->merge_tok.data(), sizeof(int32_t) * p->merge_tok.size());
      fill(o.single_tok, p->single_tok.data(), sizeof(int32_t) * p->single_tok.size());
      fill(o.tile_lm, p->tile_lm.data(), sizeof(float) * p->tile_lm.size());
      fill(o.part_lm, p->part_lm.data(), sizeof(float) * p->part_lm.size());
      fill(o.prior_rows, p->prior_rows.data(), sizeof(int32_t) * p->prior_rows.size());
      fill(o.merge_fix, p->merge_fix.data(), sizeof(int32_t) * p->merge_fix.size());
    }
  } catch (const std::bad_alloc&) {
    rc = TL_ENOMEM;
    set_error("tl_plan_create: host allocation failed");
  }
  if (rc != TL_OK) {
    delete p;
    return rc;
  }
  *out = p;
  return TL_OK;
}

tl_status tl_plan_destroy(tl_plan* plan) {
  if (!plan) return TL_OK;
  if (plan->blob_dev) (void)hipFree(plan->blob_dev);
  delete plan;
  return TL_OK;
}

tl_status tl_plan_get_info(const tl_plan* plan, tl_plan_info* info) {
  if (!plan || !info) TL_FAIL(TL_EINVAL, "tl_plan_get_info: bad argument");
  *info = plan->info;
  return TL_OK;
}

tl_status tl_plan_hot_slots(const tl_plan* plan, int32_t max_n, int32_t* slots_out, int64_t* loads_out, int32_t* n_out) {
  if (!plan || max_n < 0 || !n_out || (max_n > 0 && !slots_out)) TL_FAIL(TL_EINVAL, "tl_plan_hot_slots: bad argument");
  // Best-first search from the root over the nodes this batch walked: a node enters the frontier when
  // its parent leaves it and is never more loaded than its parent, so nodes leave in order of
  // decreasing load (equal loads: first visited first) and only the children of what is returned
  // are ever looked at.
  int32_t n = 0;
  try {
    auto later = [&](int32_t a, int32_t b) { return plan->bt_load[a] != plan->bt_load[b] ? plan->bt_load[a] < plan->bt_load[b] : a > b; };
    std::priority_queue<int32_t, std::vector<int32_t>, decltype(later)> frontier(later);
    for (int32_t c : plan->bt_roots) frontier.push(c);
    while (n < max_n && !frontier.empty()) {
      const int32_t x = frontier.top();
      frontier.pop();
      slots_out[n] = plan->bt_slot[x];
      if (loads_out) loads_out[n] = plan->bt_load[x];
      ++n;
      for (int32_t c = plan->bt_first_child[x]; c >= 0; c = plan->bt_next_sib[c]) frontier.push(c);
    }
  } catch (const std::bad_alloc&) {
    TL_FAIL(TL_ENOMEM, "tl_plan_hot_slots: host allocation failed");
  }
  *n_out = n;
  return TL_OK;
}

tl_status tl_plan_export_sizes(const tl_plan* plan, int32_t* n_item_tokens, int32_t* n_item_slots) {
  if (!plan) TL_FAIL(TL_EINVAL, "tl_plan_export_sizes: null plan");
  if (n_item_tokens) *n_item_tokens = (int32_t)plan->item_tokens.size();
  if (n_item_slots) *n_item_slots = (int32_t)plan->item_slots.size();
  return TL_OK;
}

tl_status tl_plan_export(const tl_plan* plan, int32_t* item_row_base, int32_t* item_tok_ptr, int32_t* item_tokens,
                         int32_t* item_slot_ptr, int32_t* item_slots, int32_t* merge_ptr, int32_t* merge_rows) {
  if (!plan) TL_FAIL(TL_EINVAL, "tl_plan_export: null plan");
  auto cp = [](int32_t* dst, const std::vector<int32_t>& src) {
    if (dst && !src.empty()) memcpy(dst, src.data(), sizeof(int32_t) * src.size());
  };
  cp(item_row_base, plan->item_row_base);
  cp(item_tok_ptr, plan->item_tok_ptr);
  cp(item_tokens, plan->item_tokens);
  cp(item_slot_ptr, plan->item_slot_ptr);
  cp(item_slots, plan->item_slots);
  cp(merge_ptr, plan->merge_ptr);
  cp(merge_rows, plan->merge_rows);
  return TL_OK;
}

}  // extern "C"

namespace tl {

tl_status plan_device_ready(tl_plan* p, hipStream_t stream) {
  if (p->blob_dev) return TL_OK;
  void* blob = nullptr;
  TL_HIP(hipMalloc(&blob, p->blob_host.size()));
  // on the caller's stream, in order with the kernels that read it; the host block belongs to the
  // plan, which the caller keeps alive until the stream work of its calls has completed
  hipError_t e = hipMemcpyAsync(blob, p->blob_host.data(), p->blob_host.size(), hipMemcpyHostToDevice, stream);
  if (e != hipSuccess) {
    (void)hipFree(blob);
    TL_FAIL(TL_EHIP, "plan upload failed: %s", hipGetErrorString(e));
  }
  p->blob_dev = blob;
  return TL_OK;
}

tl_status plan_is_current(const tl_plan* plan, const tl_pool* pool, const char* who) {
  if (plan->pool != pool) TL_FAIL(TL_EINVAL, "%s: plan was built for another pool", who);
  if (plan->pool_generation != pool->generation)
    TL_FAIL(TL_EINVAL, "%s: the pool has changed since the plan was built (put, append, adopt or evict): build a new plan", who);
  return TL_OK;
}

}  // namespace tl
