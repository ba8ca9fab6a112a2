// Extend work planner (host).
//
// Work unit: one query tile (block_m packed rows of one sequence and kv head)
// over a contiguous range of keys.  A tile whose rows end at token t_last needs
// keys [0, Lp + t_last + 1) (bottom-right causal).  When there are too few
// tiles to fill the GPU, each tile's key range is split into chunks of about
// equal length ("split-K"); the chunks write unnormalised partials that a
// second kernel merges with a log-sum-exp weighting.
//
// A plan whose workgroups would still finish far apart is levelled (level_plan).
//
// Launch order is XCD-aware: the dispatcher hands workgroup i to XCD i % X, and
// each XCD has its own L2.  All tiles of one (sequence, kv head) read the same
// keys, so the work of a (sequence, kv head) that fills whole rounds of the GPU
// is dealt round by round across all XCDs (every XCD streams the same keys at
// the same time), and the rest of it is kept on one XCD (split into several
// bundles only when there are fewer bundles than XCDs), bundles spread over
// XCDs longest-processing-time first; the per-XCD queues are interleaved.
// Queues that run out early are padded with idle items so that later items
// still land on their XCD.
#include "planner.h"

#include <algorithm>
#include <climits>
#include <iterator>
#include <numeric>

namespace cw {
namespace {

constexpr int32_t MIN_CHUNK_TILES = 4;  // a chunk of fewer keys wastes the Q load

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct Tile {
  int32_t seq, kvh, q_row0, rows, kv_len, n_kt, n_pre;  // n_pre: key tiles wholly in the prefix
};

// Work of one (sequence, kv head), or a share of it: items [first, first + n) of
// the plan's items in bundle order.
struct Bundle {
  int64_t first = 0, n = 0;
  int64_t cost = 0;  // key tiles
};

int64_t key_tiles(const WorkItem& w) { return (w.kv_end - w.kv_begin + BLOCK_N - 1) / BLOCK_N; }

void layout_workspace(ExtendPlan& plan, int32_t head_dim);

size_t plan_meta_bytes(size_t n_seqs, size_t n_items, size_t n_groups) {
  return align256(align256(align256(n_seqs * sizeof(SeqInfo)) + n_items * sizeof(WorkItem)) +
                  n_groups * sizeof(CombineGroup));
}

// Entries of the launch list made of these queues: they are interleaved, short ones
// padded with idle items, without trailing idle items (one used queue: as it is).
template <class T>
size_t launch_count(const std::vector<std::vector<T>>& queues) {
  size_t longest = 0, last = 0, used = 0;
  for (size_t x = 0; x < queues.size(); ++x) {
    used += queues[x].empty() ? 0 : 1;
    if (queues[x].size() >= longest) {
      longest = queues[x].size();
      last = x;
    }
  }
  return used > 1 ? (longest - 1) * queues.size() + last + 1 : longest;
}

// ---- levelled plans -------------------------------------------------------
// The cost model, in hundredths of the time one workgroup takes for a prefix
// key tile when all its rows are in use (1.7-2.2 us at head dim 128).  Fewer
// rows make a tile cheaper only down to the time its K/V take to arrive
// (measured per tile, 256 workgroups, unshared K/V: 2.19 us with 256 rows, 1.94
// with 192, 1.58 with 128, 1.53 with 32).  At head dim 64 the same units stand for
// about half that time.  A tile past the prefix counts suffix_weight: right for one
// that straddles the prefix's end or the diagonal, too much for one wholly among the
// new tokens, which the kernel runs without masks like a prefix tile.
constexpr int64_t kItemCost = 300;       // start-up and epilogue of a work item
constexpr int64_t kMergeCost = 450;      // the merge kernel's launch and latency
constexpr int64_t kMergePartCost = 2;    // per partial slot merged
constexpr int64_t kMinGap = MIN_CHUNK_TILES * 100 + kItemCost;
// What cutting tiles has to gain at least (about 55 us at head dim 128): calls of
// 20-100 us lost 5-60 us to the merge and the larger plan when they were levelled.
// Asked in full also of plans that have partials, and so a merge, already.
constexpr int64_t kMinCutGain = 3000;

int64_t row_rate(int32_t rows) {
  constexpr int64_t rate[8] = {72, 72, 72, 72, 80, 89, 95, 100};
  return rate[std::min(7, (rows - 1) / 32)];
}

// Key tiles [a, b) of a query tile.
int64_t span_cost(const Tile& t, int64_t a, int64_t b, int64_t suffix_weight) {
  const int64_t pre = std::max<int64_t>(0, std::min<int64_t>(b, t.n_pre) - a), suf = (b - a) - pre;
  return (pre * 100 + suf * suffix_weight) * row_rate(t.rows) / 100;
}
int64_t tile_cost(const Tile& t, int64_t suffix_weight) {
  return kItemCost + span_cost(t, 0, t.n_kt, suffix_weight);
}
// The last key tile up to which the tiles from `a` on cost at most `budget`.
int64_t span_end(const Tile& t, int64_t a, int64_t budget, int64_t suffix_weight) {
  const int64_t units = std::max<int64_t>(0, budget) * 100 / row_rate(t.rows);
  const int64_t pre = std::max<int64_t>(0, t.n_pre - a);
  if (units < pre * 100) return a + units / 100;
  return a + pre + (units - pre * 100) / suffix_weight;
}

// Workgroup slots by the time they are free: a binary heap, soonest first.
struct Slots {
  struct Slot {
    int64_t t;
    int32_t r;
    bool operator<(const Slot& o) const { return t != o.t ? t < o.t : r < o.r; }
  };
  std::vector<Slot> s;
  explicit Slots(int64_t R) : s(static_cast<size_t>(R)) {
    for (int64_t r = 0; r < R; ++r) s[r] = Slot{0, static_cast<int32_t>(r)};
  }
  int64_t soonest() const { return s[0].t; }
  void take(int64_t cost) {  // the soonest slot runs for `cost` more
    Slot v = s[0];
    v.t += cost;
    size_t i = 0;
    for (;;) {
      size_t c = 2 * i + 1;
      if (c >= s.size()) break;
      if (c + 1 < s.size() && s[c + 1] < s[c]) ++c;
      if (!(s[c] < v)) break;
      s[i] = s[c];
      i = c;
    }
    s[i] = v;
  }
  int64_t latest() const {
    int64_t m = 0;
    for (const Slot& v : s) m = std::max(m, v.t);
    return m;
  }
};

// The time at which the last of R slots finishes when the items (their costs in
// launch order) each go to the slot that is free first.
int64_t list_makespan(const std::vector<int64_t>& costs, int64_t R) {
  Slots sl(R);
  for (const int64_t c : costs) sl.take(c);
  return sl.latest();
}

struct Piece {  // key tiles [k0, k1) of tile `tile`, planned to start at `start`
  int32_t tile, k0, k1;
  int64_t start;
};
struct Left {  // a tile not placed yet, from key tile k0 on
  int32_t tile, k0;
};

// Fills the slots (in order of the time they are free) up to `level` with `left`
// in pieces of key ranges; returns the entries used up.
size_t fill_slots(const std::vector<Tile>& tiles, std::vector<Left>& left, std::vector<Slots::Slot>& slots,
                  size_t& next, int64_t level, int64_t wgt, std::vector<Piece>& out) {
  size_t i = 0;
  while (i < left.size() && next < slots.size()) {
    Slots::Slot& sl = slots[next];
    Left& l = left[i];
    const Tile& t = tiles[l.tile];
    const int64_t gap = level - sl.t;
    const int64_t whole = kItemCost + span_cost(t, l.k0, t.n_kt, wgt);
    if (whole <= gap) {
      out.push_back(Piece{l.tile, l.k0, t.n_kt, sl.t});
      sl.t += whole;
      ++i;
      continue;
    }
    if (gap >= kMinGap) {
      const int64_t e = std::min<int64_t>(span_end(t, l.k0, gap - kItemCost, wgt), t.n_kt - MIN_CHUNK_TILES);
      if (e - l.k0 >= MIN_CHUNK_TILES) {
        out.push_back(Piece{l.tile, l.k0, static_cast<int32_t>(e), sl.t});
        l.k0 = static_cast<int32_t>(e);
      }
    }
    ++next;
  }
  return i;
}

// Spreads the tiles over the queues so that each queue's R slots finish by
// `level`: a queue takes whole tiles in the order of `owned` while they end by
// `level`; what is left fills the slots in pieces of key ranges, its own queue's
// slots first.  Returns false if something does not fit.
bool level_queues(const std::vector<Tile>& tiles, const std::vector<std::vector<int32_t>>& owned,
                  const std::vector<bool>& as_before, int64_t wgt, int64_t R, int64_t level,
                  std::vector<std::vector<Piece>>& queues) {
  const size_t X = owned.size();
  std::vector<std::vector<Slots::Slot>> slots(X);
  std::vector<std::vector<Left>> left(X);
  std::vector<int32_t> pos(tiles.size());  // of a tile in its queue's `owned`
  std::vector<size_t> next(X, 0);
  queues.assign(X, {});
  for (size_t x = 0; x < X; ++x) {
    for (size_t i = 0; i < owned[x].size(); ++i) pos[owned[x][i]] = static_cast<int32_t>(i);
    if (as_before[x]) {  // tiles shaped like the queue's before: the same pieces of its own tiles
      slots[x] = slots[x - 1];
      next[x] = next[x - 1];
      for (const Piece& p : queues[x - 1])
        queues[x].push_back(Piece{owned[x][pos[p.tile]], p.k0, p.k1, p.start});
      for (const Left& l : left[x - 1]) left[x].push_back(Left{owned[x][pos[l.tile]], l.k0});
      continue;
    }
    Slots heap(R);
    for (const int32_t ti : owned[x]) {
      const int64_t c = tile_cost(tiles[ti], wgt);
      if (heap.soonest() + c > level) {
        left[x].push_back(Left{ti, 0});
        continue;
      }
      queues[x].push_back(Piece{ti, 0, tiles[ti].n_kt, heap.soonest()});
      heap.take(c);
    }
    slots[x] = std::move(heap.s);
    std::sort(slots[x].begin(), slots[x].end());
    const size_t used = fill_slots(tiles, left[x], slots[x], next[x], level, wgt, queues[x]);
    left[x].erase(left[x].begin(), left[x].begin() + static_cast<std::ptrdiff_t>(used));
  }
  std::vector<Left> rest;
  for (size_t x = 0; x < X; ++x) rest.insert(rest.end(), left[x].begin(), left[x].end());
  for (size_t x = 0; x < X && !rest.empty(); ++x) {
    const size_t used = fill_slots(tiles, rest, slots[x], next[x], level, wgt, queues[x]);
    rest.erase(rest.begin(), rest.begin() + static_cast<std::ptrdiff_t>(used));
  }
  return rest.empty();
}

// Replaces `queues` (work items per XCD in launch order) and the plan's merge
// groups where the workgroups of the plan as it is would finish far apart:
//  - by whole tiles in another order, bundles with the longest tiles first, so
//    that short tiles are left for the end (where a bundle's own tiles differ by
//    more than half, as without a cached prefix, its longest tiles first);
//  - or by that order cut off at a common level, the rest cut into key ranges that
//    fill every slot up to it.  The cuts of a bundle's tiles lie at different
//    keys, so their workgroups share less of the K/V in their XCD's L2: hence
//    whole tiles wherever they fit.
// Measured: 7 turns of 383-3506 tokens 7.90 -> 6.88 ms, 32 chunks + 32 decodes
// 4.16 -> 4.03 ms, a mixed fp8 step 5.53 -> 5.34 ms, 10 replies of 12-600 tokens
// 744 -> 686 us, 4 prompts of 2-6k tokens without a prefix 365 -> 343 us (order
// alone).  The gain is about half of what the model says: workgroups that share
// the chip with idle CUs run faster.  The pieces' partials are fp32 (their sums would
// stay in registers without the cut): rounded to bf16 they raised the error of 10
// replies against 64 bits by 1%, and in fp32 the times are the same (10 replies 688
// against 693 us, the mixed steps within 2%).
void level_plan(ExtendPlan& plan, const std::vector<Tile>& tiles, const std::vector<Bundle>& whole_bundles,
                int64_t wgt, int64_t R, int32_t head_dim, std::vector<std::vector<WorkItem>>& queues) {
  const size_t X = queues.size();
  if (tiles.empty() || tiles.size() > size_t(kMaxLevelTiles)) return;

  // the plan as it is
  int64_t now = 0, sum = 0;
  {
    std::vector<int64_t> costs, last;
    int64_t last_span = 0;
    for (const auto& q : queues) {
      costs.clear();
      for (const WorkItem& w : q) {
        Tile t{};
        t.rows = w.rows;
        t.n_pre = plan.seqs[w.seq].lp / BLOCK_N;
        costs.push_back(kItemCost + span_cost(t, w.kv_begin / BLOCK_N, (w.kv_end + BLOCK_N - 1) / BLOCK_N, wgt));
        sum += costs.back();
      }
      if (costs != last) {
        last_span = list_makespan(costs, R);
        last.swap(costs);
      }
      now = std::max(now, last_span);
    }
  }
  if (plan.n_parts > 0) now += kMergeCost + kMergePartCost * plan.n_parts;
  const int64_t slots = static_cast<int64_t>(X) * R;
  if (sum / slots * 103 >= now * 100) return;

  // bundles to queues: largest first to the least loaded queue; then, in a queue,
  // bundles with the longest tiles first
  struct Bd {
    int32_t t0, n;
    int64_t cost, longest, shortest;
  };
  std::vector<Bd> bundles;
  bundles.reserve(whole_bundles.size());
  int64_t total = 0;
  for (const Bundle& wb : whole_bundles) {
    Bd bd{static_cast<int32_t>(wb.first), static_cast<int32_t>(wb.n), 0, 0, INT64_MAX};
    for (int32_t i = bd.t0; i < bd.t0 + bd.n; ++i) {
      const int64_t c = tile_cost(tiles[i], wgt);
      bd.cost += c;
      bd.longest = std::max(bd.longest, c);
      bd.shortest = std::min(bd.shortest, c);
    }
    total += bd.cost;
    bundles.push_back(bd);
  }
  std::stable_sort(bundles.begin(), bundles.end(), [](const Bd& a, const Bd& c) { return a.cost > c.cost; });
  std::vector<std::vector<const Bd*>> mine(X);
  std::vector<int64_t> load(X, 0);
  for (const Bd& bd : bundles) {
    const size_t x = static_cast<size_t>(std::min_element(load.begin(), load.end()) - load.begin());
    load[x] += bd.cost;
    mine[x].push_back(&bd);
  }
  std::vector<std::vector<int32_t>> owned(X);
  // queue x's tiles are shaped like queue x - 1's, one by one, so the same key ranges level it
  // (equal costs would not do: a full tile and a longer one of fewer rows may cost the same)
  std::vector<bool> as_before(X, false);
  auto shaped_alike = [&](int32_t a, int32_t c) {
    return tiles[a].n_kt == tiles[c].n_kt && tiles[a].n_pre == tiles[c].n_pre && tiles[a].rows == tiles[c].rows;
  };
  std::vector<int64_t> costs, last;
  int64_t ordered = 0, last_span = 0;
  for (size_t x = 0; x < X; ++x) {
    std::stable_sort(mine[x].begin(), mine[x].end(),
                     [](const Bd* a, const Bd* c) { return a->longest > c->longest; });
    costs.clear();
    for (const Bd* bd : mine[x]) {
      const bool reverse = bd->shortest * 2 < bd->longest;
      for (int32_t i = 0; i < bd->n; ++i) {
        owned[x].push_back(reverse ? bd->t0 + bd->n - 1 - i : bd->t0 + i);
        costs.push_back(tile_cost(tiles[owned[x].back()], wgt));
      }
    }
    as_before[x] = x > 0 && std::equal(owned[x].begin(), owned[x].end(), owned[x - 1].begin(), owned[x - 1].end(),
                                       shaped_alike);
    if (costs != last) {
      last_span = list_makespan(costs, R);
      last.swap(costs);
    }
    ordered = std::max(ordered, last_span);
  }
  const bool reorder = ordered * 104 < now * 100;
  const int64_t best = reorder ? ordered : now;

  // the lowest level that holds everything (each cut adds an item's own cost)
  std::vector<std::vector<Piece>> pieces;
  std::vector<int32_t> n_of(tiles.size(), 1);
  const int64_t base = (total + slots - 1) / slots;
  bool cut = false;
  if ((base + kMergeCost) * 103 < best * 100 && best - base - kMergeCost >= kMinCutGain) {
    int64_t level = 0;
    for (int64_t k = 1; k <= 6 && !cut; ++k) {
      level = base + k * (base / 100 + kItemCost / 4);
      cut = level_queues(tiles, owned, as_before, wgt, R, level, pieces);
    }
    if (cut) {
      std::fill(n_of.begin(), n_of.end(), 0);
      for (const auto& q : pieces)
        for (const Piece& p : q) ++n_of[p.tile];
      int64_t n_parts = 0;
      size_t n_cut = 0;
      for (const int32_t n : n_of) {
        n_parts += n > 1 ? n : 0;
        n_cut += n > 1 ? 1 : 0;
      }
      const int64_t then = level + kMergeCost + kMergePartCost * n_parts;
      const int64_t slot_bytes = int64_t(plan.part_rows) * (head_dim * 4 + 8);
      const int64_t total_bytes =
          static_cast<int64_t>(plan_meta_bytes(plan.seqs.size(), launch_count(pieces), n_cut)) + n_parts * slot_bytes;
      cut = then * 103 < best * 100 && best - then >= kMinCutGain && total_bytes <= kLevelTotalBytes;
    }
  }
  if (!cut && !reorder) return;
  if (!cut) {
    std::fill(n_of.begin(), n_of.end(), 1);
    pieces.assign(X, {});
    for (size_t x = 0; x < X; ++x)
      for (const int32_t ti : owned[x]) pieces[x].push_back(Piece{ti, 0, tiles[ti].n_kt, 0});
  }
  size_t n_groups = 0;
  for (const int32_t n : n_of) n_groups += n > 1 ? 1 : 0;
  if (plan_meta_bytes(plan.seqs.size(), launch_count(pieces), n_groups) > plan.whole_meta_bytes + kLevelMetaBytes) return;

  // partial slots: a tile's pieces in key order
  plan.part_f32 = true;
  plan.groups.clear();
  plan.n_parts = 0;
  std::vector<int32_t> part0(tiles.size(), -1);
  for (size_t i = 0; i < tiles.size(); ++i) {
    if (n_of[i] < 2) continue;
    const Tile& t = tiles[i];
    part0[i] = static_cast<int32_t>(plan.n_parts);
    plan.groups.push_back(CombineGroup{t.seq, t.kvh, t.q_row0, t.rows, part0[i], n_of[i], 0, 0});
    plan.n_parts += n_of[i];
  }
  std::vector<std::pair<int32_t, int32_t>> cuts;  // (tile, first key tile) of the pieces of cut tiles
  for (const auto& q : pieces)
    for (const Piece& p : q)
      if (n_of[p.tile] > 1) cuts.emplace_back(p.tile, p.k0);
  std::sort(cuts.begin(), cuts.end());  // in tile order: a tile's first entry is at its part0
  for (size_t x = 0; x < X; ++x) {
    std::stable_sort(pieces[x].begin(), pieces[x].end(),
                     [](const Piece& a, const Piece& c) { return a.start < c.start; });
    queues[x].clear();
    queues[x].reserve(pieces[x].size());
    for (const Piece& p : pieces[x]) {
      const Tile& t = tiles[p.tile];
      int32_t part = -1;
      if (n_of[p.tile] > 1)
        part = static_cast<int32_t>(std::lower_bound(cuts.begin() + part0[p.tile], cuts.end(),
                                                     std::make_pair(p.tile, p.k0)) - cuts.begin());
      queues[x].push_back(WorkItem{t.seq, t.kvh, t.q_row0, p.k0 * BLOCK_N,
                                   std::min(p.k1 * BLOCK_N, t.kv_len), part, t.rows, 0});
    }
  }
}

}  // namespace

ExtendPlan build_extend_plan(const int32_t* prefix_lens, const int32_t* suffix_lens,
                             int32_t num_seqs, int32_t num_kv_heads, int32_t gqa_group,
                             int32_t head_dim, int32_t block_m, int32_t wgs_per_cu,
                             int32_t num_cus, int32_t num_xcds, const Tuning& tuning,
                             const int32_t* cu_rows, const int32_t* bt_rows) {
  ExtendPlan plan;
  plan.part_rows = block_m;
  plan.seqs.resize(num_seqs);
  int64_t cu = 0, n_tiles = 0;
  for (int32_t b = 0; b < num_seqs; ++b) {
    plan.seqs[b] = SeqInfo{prefix_lens[b], suffix_lens[b],
                           cu_rows ? cu_rows[b] : static_cast<int32_t>(cu), bt_rows ? bt_rows[b] : b};
    cu += suffix_lens[b];
    n_tiles += (int64_t(suffix_lens[b]) * gqa_group + block_m - 1) / block_m * num_kv_heads;
  }

  // 1. query tiles, bundle by bundle (the tiles of one sequence and kv head)
  std::vector<Tile> tiles;
  std::vector<Bundle> tile_bundles;
  tiles.reserve(static_cast<size_t>(n_tiles));
  int64_t total_kt = 0;
  for (int32_t b = 0; b < num_seqs; ++b) {
    const int64_t rows = int64_t(suffix_lens[b]) * gqa_group;
    for (int32_t h = 0; rows > 0 && h < num_kv_heads; ++h) {
      tile_bundles.push_back(Bundle{static_cast<int64_t>(tiles.size()), (rows + block_m - 1) / block_m, 0});
      for (int64_t r0 = 0; r0 < rows; r0 += block_m) {
        const int32_t nr = static_cast<int32_t>(std::min<int64_t>(block_m, rows - r0));
        const int64_t t_last = (r0 + nr - 1) / gqa_group;
        const int32_t kv_len = static_cast<int32_t>(prefix_lens[b] + t_last + 1);
        const int32_t n_kt = (kv_len + BLOCK_N - 1) / BLOCK_N;
        tiles.push_back(Tile{b, h, static_cast<int32_t>(r0), nr, kv_len, n_kt,
                             std::min(n_kt, prefix_lens[b] / BLOCK_N)});
        total_kt += n_kt;
      }
    }
  }

  // 2. split-K: number of chunks per tile.  Automatic: when there are fewer
  // tiles than `target` workgroups (all resident at once), each tile gets
  // about n_kt / (total_kt / target) chunks, so chunks are of about equal
  // length and their count is close to the target.
  const int64_t target =
      tuning.target_wgs > 0 ? tuning.target_wgs : int64_t(std::max(1, wgs_per_cu)) * num_cus;
  double chunk_len = 0.0;  // 0: no split
  if (tuning.kv_chunk_tiles > 0) {
    chunk_len = tuning.kv_chunk_tiles;
  } else if (static_cast<int64_t>(tiles.size()) < target && !tiles.empty()) {
    chunk_len = std::max<double>(MIN_CHUNK_TILES, double(total_kt) / double(target));
  }
  auto n_chunks = [&](int32_t n_kt) -> int64_t {
    if (chunk_len <= 0.0) return 1;
    if (tuning.kv_chunk_tiles > 0) return std::max<int64_t>(1, (n_kt + tuning.kv_chunk_tiles - 1) / tuning.kv_chunk_tiles);
    const int64_t n = static_cast<int64_t>(double(n_kt) / chunk_len + 0.5);
    return std::max<int64_t>(1, std::min<int64_t>(n, n_kt / MIN_CHUNK_TILES));
  };

  // 3. work items, bundle by bundle, a bundle's first chunks before its second ones
  std::vector<WorkItem> items;
  std::vector<Bundle> bundles;
  std::vector<int64_t> first;  // of the bundle's tiles: first key tile of each chunk, and the end
  std::vector<std::pair<int64_t, int32_t>> chunk_at;  // of each tile: where its chunks start in `first`; part0
  items.reserve(tiles.size());
  bundles.reserve(tile_bundles.size());
  for (const Bundle& tb : tile_bundles) {
    Bundle bd{static_cast<int64_t>(items.size()), 0, 0};
    first.clear();
    chunk_at.clear();
    int64_t most = 1;
    for (int64_t ti = tb.first; ti < tb.first + tb.n; ++ti) {
      const Tile& t = tiles[ti];
      const int64_t n_c = n_chunks(t.n_kt);
      most = std::max(most, n_c);
      int32_t part0 = -1;
      if (n_c > 1) {
        part0 = static_cast<int32_t>(plan.n_parts);
        plan.groups.push_back(CombineGroup{t.seq, t.kvh, t.q_row0, t.rows, part0,
                                           static_cast<int32_t>(n_c), 0, 0});
        plan.n_parts += n_c;
      }
      chunk_at.emplace_back(static_cast<int64_t>(first.size()), part0);
      // chunk boundaries: equal shares of the tile's cost, a key tile that
      // reaches past the cached prefix (read from the new tokens) counting
      // suffix_weight / 100 of a prefix tile (forced chunk sizes: equal key
      // counts); every chunk at least one tile long
      const int64_t n_pre = t.n_pre;
      const int64_t wgt = tuning.kv_chunk_tiles > 0 ? 100 : std::max(1, tuning.suffix_weight);
      const int64_t total_cost = n_pre * 100 + (t.n_kt - n_pre) * wgt;
      first.push_back(0);
      for (int64_t c = 1; c < n_c; ++c) {
        int64_t b = c * t.n_kt / n_c;
        if (wgt != 100) {
          const int64_t goal = c * total_cost / n_c;
          b = goal <= n_pre * 100 ? (goal + 99) / 100 : n_pre + (goal - n_pre * 100 + wgt - 1) / wgt;
        }
        first.push_back(std::min(std::max(b, first.back() + 1), t.n_kt - (n_c - c)));
      }
      first.push_back(t.n_kt);
    }
    for (int64_t c = 0; c < most; ++c)
      for (int64_t i = 0; i < tb.n; ++i) {
        const Tile& t = tiles[tb.first + i];
        const int64_t at = chunk_at[i].first;
        const int64_t end = i + 1 < tb.n ? chunk_at[i + 1].first : static_cast<int64_t>(first.size());
        if (at + c + 1 >= end) continue;
        const int64_t kt0 = first[at + c], kt1 = first[at + c + 1];
        const int32_t part0 = chunk_at[i].second;
        items.push_back(WorkItem{t.seq, t.kvh, t.q_row0, static_cast<int32_t>(kt0 * BLOCK_N),
                                 static_cast<int32_t>(std::min<int64_t>(kt1 * BLOCK_N, t.kv_len)),
                                 part0 >= 0 ? part0 + static_cast<int32_t>(c) : -1, t.rows, 0});
        bd.cost += key_tiles(items.back());
      }
    bd.n = static_cast<int64_t>(items.size()) - bd.first;
    bundles.push_back(bd);
  }
  auto recount = [&](Bundle& bd) {
    bd.cost = 0;
    for (int64_t i = bd.first; i < bd.first + bd.n; ++i) bd.cost += key_tiles(items[i]);
  };

  // 4. Bundles that fill whole rounds of the GPU (R items per XCD, one per
  // resident workgroup slot): dealt across every XCD a round at a time, so all
  // XCDs stream the keys of the same (sequence, kv head) at once and what one
  // XCD's L2 has dropped is still in the memory-side cache for the others (a
  // bundle kept on one XCD for several rounds has all XCDs streaming different
  // heads, more than that cache holds).  The items of every other round run in
  // reverse order, so the slot that drew a short tile draws a long one next and
  // the slots of an XCD stay close together in the key stream.  Within a round
  // each XCD takes consecutive items (tiles of about equal length), rotating
  // over the round's blocks from one round to the next.
  const int32_t X = std::max(1, num_xcds);
  const int64_t R = std::max<int64_t>(1, int64_t(std::max(1, wgs_per_cu)) * num_cus / X);
  std::vector<std::vector<WorkItem>> queues(X);
  bool dealt = false;
  if (tuning.deal_rounds != 0) {
    int64_t round = 0;
    for (auto& bd : bundles) {
      const int64_t n_rounds = bd.n / (R * X);
      for (int64_t r = 0; r < n_rounds; ++r, ++round)
        for (int32_t x = 0; x < X; ++x) {
          // XCD x takes block (x + round) % X of the round's X blocks of R
          // items: blocks later in a bundle hold longer tiles (more keys), and
          // the rotation gives every XCD each position in turn
          const auto b0 = items.begin() + bd.first + (r * X + (x + round) % X) * R;
          if (round & 1) queues[x].insert(queues[x].end(), std::make_reverse_iterator(b0 + R),
                                          std::make_reverse_iterator(b0));
          else queues[x].insert(queues[x].end(), b0, b0 + R);
        }
      if (n_rounds > 0) {
        dealt = true;
        bd.first += n_rounds * R * X;
        bd.n -= n_rounds * R * X;
        recount(bd);
      }
    }
    bundles.erase(std::remove_if(bundles.begin(), bundles.end(), [](const Bundle& b) { return b.n == 0; }),
                  bundles.end());
  }

  // 5. enough bundles to occupy every XCD: halve the largest while possible
  while (static_cast<int32_t>(bundles.size()) < 2 * X) {
    auto it = std::max_element(bundles.begin(), bundles.end(),
                               [](const Bundle& a, const Bundle& c) { return a.n < c.n; });
    if (it == bundles.end() || it->n < 2) break;
    const int64_t half = it->n / 2;
    Bundle hi{it->first + half, it->n - half, 0};
    it->n = half;
    recount(*it);
    recount(hi);
    bundles.push_back(hi);
  }

  // 6. LPT assignment of the other bundles to XCD queues (after the dealt
  // rounds, which every queue holds the same number of), levelled where the
  // workgroups would finish far apart, then interleave
  std::stable_sort(bundles.begin(), bundles.end(),
                   [](const Bundle& a, const Bundle& c) { return a.cost > c.cost; });
  std::vector<int64_t> load(X, 0);
  for (auto& bd : bundles) {
    const int32_t x = static_cast<int32_t>(std::min_element(load.begin(), load.end()) - load.begin());
    load[x] += bd.cost;
    queues[x].insert(queues[x].end(), items.begin() + bd.first, items.begin() + bd.first + bd.n);
  }
  plan.whole_meta_bytes = plan_meta_bytes(plan.seqs.size(), launch_count(queues), plan.groups.size());
  if (tuning.kv_chunk_tiles == 0 && tuning.target_wgs == 0 && !dealt)
    level_plan(plan, tiles, tile_bundles, std::max(1, tuning.suffix_weight), R, head_dim, queues);
  size_t max_len = 0;
  for (auto& qv : queues) max_len = std::max(max_len, qv.size());
  const WorkItem idle{-1, 0, 0, 0, 0, -1, 0, 0};
  int32_t used_queues = 0;
  for (auto& qv : queues) used_queues += qv.empty() ? 0 : 1;
  plan.items.reserve(max_len * static_cast<size_t>(X));
  for (size_t i = 0; i < max_len; ++i)
    for (int32_t x = 0; x < X; ++x) {
      if (i < queues[x].size()) plan.items.push_back(queues[x][i]);
      else if (used_queues > 1) plan.items.push_back(idle);
    }
  // trailing idle items launch nothing useful
  while (!plan.items.empty() && plan.items.back().seq < 0) plan.items.pop_back();

  // 7. workspace layout
  layout_workspace(plan, head_dim);
  return plan;
}

namespace {
void layout_workspace(ExtendPlan& plan, int32_t head_dim) {
  plan.off_seqs = 0;
  plan.off_items = align256(plan.off_seqs + plan.seqs.size() * sizeof(SeqInfo));
  plan.off_groups = align256(plan.off_items + plan.items.size() * sizeof(WorkItem));
  plan.meta_bytes = align256(plan.off_groups + plan.groups.size() * sizeof(CombineGroup));
  for (const CombineGroup& g : plan.groups) plan.max_parts = std::max(plan.max_parts, g.n_parts);
  plan.off_part_o = plan.meta_bytes;
  // the partial O in fp32 or bf16, the running max and sum in fp32
  plan.off_part_ml =
      align256(plan.off_part_o + size_t(plan.n_parts) * plan.part_rows * head_dim * (plan.part_f32 ? 4 : 2));
  plan.total_bytes = align256(plan.off_part_ml + size_t(plan.n_parts) * plan.part_rows * 2 * sizeof(float));
}
}  // namespace

namespace {
// Items and merge groups of a decode cut into chunks of `chunk` keys.
std::pair<int64_t, int64_t> decode_counts(const int32_t* prefix_lens, int32_t num_seqs, int32_t num_kv_heads,
                                          int64_t chunk) {
  int64_t items = 0, groups = 0;
  for (int32_t b = 0; b < num_seqs; ++b) {
    const int64_t n_c = (int64_t(prefix_lens[b]) + chunk) / chunk;  // of prefix_lens[b] + 1 keys
    items += n_c;
    groups += n_c > 1 ? 1 : 0;
  }
  return {items * num_kv_heads, groups * num_kv_heads};
}

// The chunk length (keys) that fills whole rounds of the GPU.  Where one round can
// hold the call, that is the shortest chunk with at most four items per CU (three, the
// resident ones, for bf16 pools); where the longest chunk gives up to four rounds, the
// shortest with that many.  A round that is partly filled costs nearly a full one,
// because a wave alone on its CU takes about half the time per tile of one among
// three: too little to make up for the empty slots.  Measured with 8 kv heads of 128:
// bf16 pools, 8 prefixes of 2k-32k: 1072 items (1.4 rounds) 102 us, 1536 items 92 us;
// 12 of 8k-30k: 1592 items 147 us, 2296 items 132 us; 16 of 1k-16k: 824 items 82 us, 728
// items 76 us.  fp8 pools, 2 of 30k-50k: 1512 items (six per CU) 37.4 us, 984 items 33.0
// us, 760 items 33.2 us; 4 of 20k-60k: 1080 items 61 us, 1520 items 54 us; 24 of 3k-20k:
// 1984 items 108 us, 2976 items 94 us.  Beyond four rounds the longest chunk is best
// (48 decodes over fp8 pages: 6464 items 278 us, 7400 items 280 us).  Where more than
// half of the items are the last, shorter chunks of their sequences, no chunk length
// makes them even, and `plain` stays (96 prefixes of 200-6000 keys, 64-wide heads: 107 us
// with it, 111-117 us with 1100-1500 items).  The figures are from bf16 partials; those
// of an adjusted plan are fp32 (ExtendPlan::part_f32), which takes up to 2.7 us more and
// leaves it ahead of the plain chunk: 8 bf16 prefixes of 2k-32k 100.3 us plain, 94.2 us
// adjusted with bf16 partials, 96.5 us with fp32 ones; 16 of 1k-16k 99.9, 91.8, 93.9 us;
// fp8, 24 of 3k-20k 106.4, 100.0, 102.7 us.  Error against 64 bits of two fp8 decodes:
// 2.48e-3 plain, 2.79e-3 adjusted with bf16 partials, 2.19e-3 with fp32 ones.
int64_t round_chunk(const int32_t* prefix_lens, int32_t num_seqs, int32_t num_kv_heads, int64_t unit,
                    int64_t max_chunk, int64_t min_chunk, int64_t num_cus, int64_t waves_per_cu, int64_t plain) {
  auto items = [&](int64_t chunk) { return decode_counts(prefix_lens, num_seqs, num_kv_heads, chunk).first; };
  const int64_t slots = num_cus * waves_per_cu, one_round = num_cus * std::min<int64_t>(waves_per_cu, 4);
  const int64_t longest = max_chunk / unit * unit;
  const int64_t least = items(longest);
  int64_t most = std::max(one_round, least);  // (2% over: 1040 items for 1024 29.5 us, 1480 items 33.8 us)
  if (least * 50 > one_round * 51) {
    const int64_t rounds = (least + slots - 1) / slots;
    if (rounds > 4) return plain;
    most = rounds * slots;
  }
  int64_t lo = min_chunk / unit, hi = longest / unit;  // items(hi) <= most; items never rise with the chunk
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (items(mid * unit) <= most) hi = mid;
    else lo = mid + 1;
  }
  const auto n = decode_counts(prefix_lens, num_seqs, num_kv_heads, lo * unit);
  const auto n_plain = decode_counts(prefix_lens, num_seqs, num_kv_heads, plain);
  if (int64_t(num_seqs) * num_kv_heads * 2 > n.first) return plain;
  // the larger work list stays within what the limits on a call's plan allow for
  if ((n.first - n_plain.first + n.second - n_plain.second + 24) * int64_t(sizeof(WorkItem)) > int64_t(kLevelMetaBytes))
    return plain;
  return lo * unit;
}
}  // namespace

// Decode planning.  The cached prefix of each (sequence, kv head) is cut into
// chunks of whole decode tiles and whole pages (at most 64 pages, the kernel
// keeps one page id per lane).  Chunks are about as long as one wave per resident
// slot allows (a decode wave streams its chunk at its share of HBM bandwidth;
// every wave pays one start-up latency for its page ids and first tile, so
// fewer, longer waves waste less), within the 64-page cap, adjusted to whole
// rounds of the GPU (round_chunk).  The new token's own key rides with the last chunk.
ExtendPlan build_decode_plan(const int32_t* prefix_lens, int32_t num_seqs, int32_t num_kv_heads,
                             int32_t gqa_group, int32_t head_dim, int32_t page_size,
                             int32_t keys_per_tile, int32_t waves_per_cu, int32_t num_cus,
                             const Tuning& tuning, size_t meta_at, const int32_t* cu_rows,
                             const int32_t* bt_rows) {
  ExtendPlan plan;
  plan.part_rows = gqa_group;
  plan.seqs.resize(num_seqs);
  int64_t total_tiles = 0;
  for (int32_t b = 0; b < num_seqs; ++b) {
    plan.seqs[b] = SeqInfo{prefix_lens[b], 1, cu_rows ? cu_rows[b] : b, bt_rows ? bt_rows[b] : b};
    total_tiles += (int64_t(prefix_lens[b]) + keys_per_tile) / keys_per_tile * num_kv_heads;
  }
  const int64_t unit = std::max<int64_t>(keys_per_tile, page_size);  // chunk granule
  const int64_t max_chunk = int64_t(64) * page_size;                 // keys
  int64_t chunk;
  if (tuning.kv_chunk_tiles > 0) {
    chunk = int64_t(tuning.kv_chunk_tiles) * keys_per_tile;
  } else {
    const int64_t target = tuning.target_wgs > 0 ? tuning.target_wgs : int64_t(num_cus) * waves_per_cu;
    const int64_t tiles = std::max<int64_t>(2, (total_tiles + target - 1) / target);
    chunk = tiles * keys_per_tile;
  }
  chunk = std::min(max_chunk, std::max(unit, (chunk + unit - 1) / unit * unit));
  const int64_t plain_chunk = chunk;
  if (tuning.kv_chunk_tiles == 0 && tuning.target_wgs == 0)
    chunk = round_chunk(prefix_lens, num_seqs, num_kv_heads, unit, max_chunk,
                        std::max<int64_t>(unit, (2 * int64_t(keys_per_tile) + unit - 1) / unit * unit), num_cus,
                        waves_per_cu, plain_chunk);
  if (chunk != plain_chunk) {
    // a plan that would fit the kernel arguments stays there: it then needs neither an
    // upload nor, when captured, any set-up (other chunks may end more sequences short)
    auto fits = [&](int64_t c) {
      size_t n_tails = 0;
      for (int32_t b = 0; b < num_seqs; ++b) n_tails += (int64_t(prefix_lens[b]) + 1) % c != 0 ? 1 : 0;
      return compact_arg_fits(
          compact_bytes(meta_at + align256(size_t(num_seqs) * sizeof(SeqInfo)), size_t(num_seqs), n_tails));
    };
    if (!fits(chunk) && fits(plain_chunk)) chunk = plain_chunk;
  }
  // Longest chunks first so that short tails fill in at the end: every chunk but
  // the last of a (sequence, kv head) has the full length, so the order is the
  // full-length chunks in build order, then the shorter last chunks by length
  // (stable), the same as a stable sort of all items by length.
  int64_t n_items = 0;
  for (int32_t b = 0; b < num_seqs; ++b) n_items += (int64_t(prefix_lens[b]) + chunk) / chunk;
  plan.items.reserve(size_t(n_items * num_kv_heads));
  std::vector<WorkItem> tails;
  tails.reserve(size_t(num_seqs) * num_kv_heads);
  for (int32_t b = 0; b < num_seqs; ++b) {
    const int64_t n = int64_t(prefix_lens[b]) + 1;  // keys including the new one
    const int64_t n_c = (n + chunk - 1) / chunk;
    for (int32_t h = 0; h < num_kv_heads; ++h) {
      int32_t part0 = -1;
      if (n_c > 1) {
        part0 = static_cast<int32_t>(plan.n_parts);
        plan.groups.push_back(CombineGroup{b, h, 0, gqa_group, part0, static_cast<int32_t>(n_c), 0, 0});
        plan.n_parts += n_c;
      }
      for (int64_t c = 0; c < n_c; ++c) {
        const WorkItem it{b, h, 0, static_cast<int32_t>(c * chunk),
                          static_cast<int32_t>(std::min(n, (c + 1) * chunk)),
                          n_c > 1 ? static_cast<int32_t>(part0 + c) : -1, gqa_group, 0};
        (it.kv_end - it.kv_begin == chunk ? plan.items : tails).push_back(it);
      }
    }
  }
  std::stable_sort(tails.begin(), tails.end(), [](const WorkItem& a, const WorkItem& c) {
    return (a.kv_end - a.kv_begin) > (c.kv_end - c.kv_begin);
  });
  plan.items.insert(plan.items.end(), tails.begin(), tails.end());
  plan.part_f32 = chunk != plain_chunk;
  layout_workspace(plan, head_dim);
  plan.whole_meta_bytes = plan.meta_bytes;
  if (chunk != plain_chunk) {
    const auto n = decode_counts(prefix_lens, num_seqs, num_kv_heads, plain_chunk);
    plan.whole_meta_bytes = plan_meta_bytes(plan.seqs.size(), static_cast<size_t>(n.first), static_cast<size_t>(n.second));
  }

  // the compact form: one record per sequence, the order of the last chunks
  plan.compact = true;
  plan.recs.resize(num_seqs);
  int32_t full_off = 0, part_off = 0, group_off = 0;
  std::vector<std::pair<int64_t, int32_t>> tail_len;  // (length, sequence)
  for (int32_t b = 0; b < num_seqs; ++b) {
    const int64_t n = int64_t(prefix_lens[b]) + 1;
    const int32_t nc = static_cast<int32_t>((n + chunk - 1) / chunk);
    const int32_t full = n % chunk == 0 ? nc : nc - 1;
    plan.recs[b] = DecodeRec{full_off, full, nc, static_cast<int32_t>(n), part_off, group_off};
    full_off += full * num_kv_heads;
    if (nc > 1) {
      part_off += nc * num_kv_heads;
      group_off += num_kv_heads;
    }
    if (full < nc) tail_len.emplace_back(n - int64_t(full) * chunk, b);
  }
  std::stable_sort(tail_len.begin(), tail_len.end(),
                   [](const std::pair<int64_t, int32_t>& a, const std::pair<int64_t, int32_t>& c) {
                     return a.first > c.first;
                   });
  for (const auto& t : tail_len) plan.tails.push_back(t.second);
  ExpandDesc& d = plan.desc;
  d.n_seqs = num_seqs;
  d.n_full = full_off;
  d.n_items = static_cast<int32_t>(plan.items.size());
  d.n_groups = static_cast<int32_t>(plan.groups.size());
  d.n_tails = static_cast<int32_t>(plan.tails.size());
  d.chunk = static_cast<int32_t>(chunk);
  d.hkv = num_kv_heads;
  d.rows = gqa_group;
  d.items_off = static_cast<uint32_t>(plan.off_items);
  d.groups_off = static_cast<uint32_t>(plan.off_groups);
  return plan;
}

void pack_plan_head(const ExtendPlan& plan, uint8_t* dst) {
  std::fill(dst, dst + plan.off_items, uint8_t(0));
  std::copy(reinterpret_cast<const uint8_t*>(plan.seqs.data()),
            reinterpret_cast<const uint8_t*>(plan.seqs.data() + plan.seqs.size()), dst + plan.off_seqs);
}

void pack_plan_meta(const ExtendPlan& plan, uint8_t* dst) {
  std::fill(dst, dst + plan.meta_bytes, uint8_t(0));
  std::copy(reinterpret_cast<const uint8_t*>(plan.seqs.data()),
            reinterpret_cast<const uint8_t*>(plan.seqs.data() + plan.seqs.size()), dst + plan.off_seqs);
  std::copy(reinterpret_cast<const uint8_t*>(plan.items.data()),
            reinterpret_cast<const uint8_t*>(plan.items.data() + plan.items.size()), dst + plan.off_items);
  std::copy(reinterpret_cast<const uint8_t*>(plan.groups.data()),
            reinterpret_cast<const uint8_t*>(plan.groups.data() + plan.groups.size()), dst + plan.off_groups);
}

}  // namespace cw
