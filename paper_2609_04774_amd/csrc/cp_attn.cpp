// Host side of the C ABI: argument checks, the per-launch work list, the
// staging of descriptors into the caller's workspace, and the launches.
//
// Work list.  Every descriptor contributes, per non-empty chunk of its rank,
// ceil(q_len / q_per_wg) query blocks times (Hkv * groups_per_kv) head
// groups.  Items are ordered longest first (visible keys per item), which
// makes the hardware's in-order workgroup dispatch an LPT schedule, and are
// interleaved so that item i lands on XCD i % 8 with all items of one KV head
// group on the same XCD (where the groups are a multiple of the XCDs, else as
// many as that order leaves): the workgroups streaming one head's K/V share
// that XCD's L2.
//
// Cut key walks.  A launch whose work items do not fill the 256 compute units
// evenly (few items, or items of very different lengths) has some of its walks
// of key tiles cut into pieces; each piece is its own workgroup and writes a
// partial result (O, LSE over its keys) to the workspace, and split_merge
// combines an item's pieces exactly (the same log-sum-exp combination as
// cp_attn_merge).
//
// Choice.  The attention kernel runs 256- or 384-row workgroups.  For each
// shape the uncut list, lists cut to a longest piece and, for long walks, the
// balance cuts are timed by a simulation of the dispatch (below), and the one
// that ends first is launched.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <atomic>
#include <chrono>
#include <mutex>
#include <numeric>
#include <queue>
#include <string>
#include <thread>
#include <vector>

#include "internal.h"

using namespace cpattn;

namespace {

constexpr int kXcds = 8;
constexpr size_t kItemsAlign = 256;

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int gcd_int(int a, int b) {
  while (b) {
    int t = a % b;
    a = b;
    b = t;
  }
  return a;
}

Shape shape_for(int Hq, int Hkv, int rows) {
  const int G = Hq / Hkv;
  Shape s;
  s.rows_per_wg = rows;
  s.heads_per_wg = gcd_int(G, 8);
  s.q_per_wg = rows / s.heads_per_wg;
  s.groups_per_kv = G / s.heads_per_wg;
  return s;
}

int check_heads(int32_t Hq, int32_t Hkv, const char* who) {
  if (Hq < 1 || Hkv < 1) return fail(CP_ERR_INVALID, std::string(who) + ": head counts must be >= 1");
  if (Hq % Hkv) return fail(CP_ERR_INVALID, std::string(who) + ": n_heads_q must be a multiple of n_heads_kv");
  if (Hq > 4096) return fail(CP_ERR_UNSUPPORTED, std::string(who) + ": more than 4096 query heads");
  return CP_OK;
}

// Validates one descriptor and converts it to the kernel's form.
int to_dev(const cp_partial_desc& x, int idx, DevDesc* out) {
  const std::string who = "cp_attn_partial: desc " + std::to_string(idx) + ": ";
  const cp_rank_plan& pl = x.plan;
  cp_rank_plan ref;
  if (make_plan(pl.prefix_len, pl.new_len, pl.C, pl.rank, &ref) != CP_OK)
    return fail(CP_ERR_INVALID, who + "plan has invalid (P, R, C, rank)");
  if (!plan_equal(ref, pl)) return fail(CP_ERR_INVALID, who + "plan does not match cp_shard_plan(P, R, C, rank)");
  if (pl.n_rows > ((int64_t)1 << 31)) return fail(CP_ERR_UNSUPPORTED, who + "more than 2^31 rows");
  const int64_t P = pl.prefix_len, R = pl.new_len;
  // The kernel walks key and query positions in 32-bit arithmetic.
  if (P + R > ((int64_t)1 << 30)) return fail(CP_ERR_UNSUPPORTED, who + "sequence beyond 2^30 tokens");
  if (x.kv_rank < CP_KV_NONE || x.kv_rank >= pl.C) return fail(CP_ERR_INVALID, who + "kv_rank out of range");
  if (x.include_prefix != 0 && x.include_prefix != 1) return fail(CP_ERR_INVALID, who + "include_prefix must be 0 or 1");
  if (x.out_order != CP_OUT_LOCAL && x.out_order != CP_OUT_SEQUENCE)
    return fail(CP_ERR_INVALID, who + "out_order must be CP_OUT_LOCAL or CP_OUT_SEQUENCE");
  if (x.reserved != 0) return fail(CP_ERR_INVALID, who + "reserved must be 0");
  if (pl.n_rows > 0) {
    if (!x.q || !x.o || !x.lse) return fail(CP_ERR_INVALID, who + "q, o and lse are required");
    if (!aligned(x.q, 16) || !aligned(x.o, 16) || !aligned(x.lse, 4))
      return fail(CP_ERR_INVALID, who + "q/o must be 16-byte and lse 4-byte aligned");
  }
  const bool use_suffix = x.kv_rank != CP_KV_NONE && R > 0;
  if (use_suffix && pl.n_rows > 0) {
    if (!x.k_new || !x.v_new) return fail(CP_ERR_INVALID, who + "k_new and v_new are required");
    if (!aligned(x.k_new, 16) || !aligned(x.v_new, 16))
      return fail(CP_ERR_INVALID, who + "k_new/v_new must be 16-byte aligned");
  }
  const bool use_prefix = x.include_prefix && P > 0;
  if (use_prefix && pl.n_rows > 0) {
    if (P % CP_KV_BLOCK_TOKENS) return fail(CP_ERR_INVALID, who + "prefix_len must be a multiple of 16 when the prefix is read");
    if (!x.k_cache || !x.v_cache || !x.block_table)
      return fail(CP_ERR_INVALID, who + "k_cache, v_cache and block_table are required");
    if (!aligned(x.k_cache, 16) || !aligned(x.v_cache, 16) || !aligned(x.block_table, 4))
      return fail(CP_ERR_INVALID, who + "k_cache/v_cache must be 16-byte and block_table 4-byte aligned");
    if (P > INT32_MAX) return fail(CP_ERR_UNSUPPORTED, who + "prefix beyond 2^31 tokens");
    if (x.n_blocks < 1) return fail(CP_ERR_INVALID, who + "n_blocks must be >= 1 when the prefix is read");
  }
  DevDesc d;
  std::memset(&d, 0, sizeof(d));
  d.q = static_cast<const uint16_t*>(x.q);
  d.k_new = static_cast<const uint16_t*>(x.k_new);
  d.v_new = static_cast<const uint16_t*>(x.v_new);
  d.k_cache = static_cast<const uint16_t*>(x.k_cache);
  d.v_cache = static_cast<const uint16_t*>(x.v_cache);
  d.block_table = x.block_table;
  d.o = x.o;
  d.lse = x.lse;
  d.P = P;
  d.R = R;
  for (int i = 0; i < 2; ++i) {
    d.q_begin[i] = pl.chunk[i].q_begin;
    d.q_len[i] = pl.chunk[i].q_len;
    d.local_off[i] = pl.chunk[i].local_offset;
    // Sequence order: the chunk's first query is suffix index q_begin - P.
    d.o_off[i] = x.out_order == CP_OUT_SEQUENCE ? pl.chunk[i].q_begin - P : pl.chunk[i].local_offset;
  }
  d.prefix_keys = use_prefix ? (int32_t)P : 0;
  // Entries are int32: a cache of more blocks than that holds every entry.
  d.n_blocks = use_prefix ? (int32_t)std::min<int64_t>(x.n_blocks, INT32_MAX) : 0;
  d.n_seg = 0;
  if (use_suffix) {
    if (x.kv_rank == CP_KV_ALL) {
      d.seg_lo[0] = P;
      d.seg_hi[0] = P + R;
      d.n_seg = 1;
    } else {
      // Rank kv_rank's own suffix keys: its chunks kv_rank and 2C-1-kv_rank.
      const int64_t s = pl.chunk_len;
      const int64_t ids[2] = {x.kv_rank, 2 * (int64_t)pl.C - 1 - x.kv_rank};
      for (int i = 0; i < 2; ++i) {
        const int64_t lo = ids[i] * s;
        const int64_t hi = std::min(R, lo + s);
        if (hi > lo) {
          d.seg_lo[d.n_seg] = P + lo;
          d.seg_hi[d.n_seg] = P + hi;
          ++d.n_seg;
        }
      }
    }
  }
  *out = d;
  return CP_OK;
}

// The last rank's chunks (C-1 and C; both of a degree of 1) follow one another,
// in the sequence and in the rank's rows: as one chunk they end in one ragged
// query block instead of two.  300 rows of 32 heads on 8 KV heads, behind 16K
// cached tokens, are 5 blocks of 64 positions, not 6: 103.1 -> 95.4 us.  (A batch
// of 64 requests, 58 of degree 1, 10835 -> 10761, is within its spread of 2 %.)
// Not with a pinned workgroup shape, whose lists keep one fixed rule, nor where
// the launch is one round without it, and faster (plan_joined).
void join_chunks(DevDesc* d) {
  if (d->q_len[1] == 0 || d->q_begin[1] != d->q_begin[0] + d->q_len[0] ||
      d->local_off[1] != d->local_off[0] + d->q_len[0] || d->o_off[1] != d->o_off[0] + d->q_len[0])
    return;
  d->q_len[0] += d->q_len[1];
  d->q_len[1] = 0;
}

constexpr int64_t kMinPieceTiles = 3;      // the shortest piece of any list: the kernel's loads run five tiles ahead
constexpr int64_t kMaxPieces = 64;
// A pinned shape (cp_set_workgroup_rows) keeps one fixed rule for launches of
// few items: pieces of at least kPinnedMinTiles, aiming at the target count.
constexpr int64_t kPinnedBelowItems = 512;
constexpr int64_t kPinnedMinTiles = 32;
constexpr int kComputeUnits = 256;         // 8 XCDs x 32 compute units
constexpr int64_t kItemSetupTiles = 16;    // a workgroup's set-up and stores, in tile times
constexpr int64_t kMinBalancePiece = 256;  // tiles of the smaller part of a balance cut
constexpr double kBalanceSlack = 1.03;

// Balance cuts.  The hardware dispatches workgroups in list order to
// whichever compute unit frees up first, so a list sorted longest first is an
// LPT schedule -- but when the long items are not a multiple of the compute
// units (384-row items of a 4096-row chunk: 344 of them for 256 units), the
// last round of long items runs on a few units while the rest idle.  This
// simulates that schedule (item time = its tiles + kItemSetupTiles) and, when
// its makespan exceeds the ideal (total / units) by more than kBalanceSlack,
// tries two ways of cutting items into pieces:
//  * fill: the same schedule, where an item that would push the least loaded
//    unit past the ideal gives that unit only the tiles that fill it up, its
//    remaining tiles going back into the queue as a later item;
//  * even: the longest items are placed whole while the least loaded unit
//    takes them within the bound; each item left that can be cut in two is
//    cut into equal pieces, m units' worth of pieces in all (m = 1 .. 4),
//    dealt in proportion to the items' lengths.
// Each candidate is scored by the schedule that the dispatch makes of it (all
// pieces sorted longest first), and the one that ends first is kept; fewer
// pieces win a tie.  Every piece keeps at least kMinBalancePiece tiles (each
// costs a set-up, and its rows a merge).  Fill suits a few long items over a
// round of shorter ones (the 32K prompt's rank 0, whose short chunk's items
// fill the gaps); even suits rounds of equally long items (a prompt behind a
// long cached prefix), where fill's remainders are too long for the room
// they find.  Returns each item's interior cut points (tile indices,
// ascending) in `cuts` (indexed by the items' numbers, allocated only when a
// cut is made), of at most max_pieces pieces.
struct ItemTiles {
  int64_t item;   // the item's number in the launch
  int64_t tiles;  // its key walk
};

// The times at which one schedule's units fall free, as a binary heap: the root
// is the first, and a unit that takes a workgroup sinks from there.
template <class T>
struct Units {
  std::vector<T> free;
  T end = 0;  // the makespan
  explicit Units(int n) : free(n, T(0)) {}
  void add(T len) {
    const T t = free[0] + len;
    const size_t n = free.size();
    size_t i = 0;
    for (size_t c = 1; c < n; c = 2 * i + 1) {
      c += c + 1 < n && free[c + 1] < free[c];
      if (free[c] >= t) break;
      free[i] = free[c];
      i = c;
    }
    free[i] = t;
    end = std::max(end, t);
  }
  // The same for the k-th workgroup of a list sorted longest first: the first of
  // each unit needs no heap (ascending times are one).
  void add_sorted(size_t k, T len) {
    if (k >= free.size()) return add(len);
    free[free.size() - 1 - k] = len;
    end = std::max(end, len);
  }
};

// Makespan of list scheduling `lens` (sorted longest first) onto units whose
// loads start at `loads`; or, as soon as it is known to exceed `give_up`,
// something above that.
int64_t list_schedule(const std::vector<int64_t>& loads, const std::vector<int64_t>& lens,
                      int64_t give_up = INT64_MAX) {
  // Of the r * n + 1 longest, some of n units takes r + 1: the shortest r + 1
  // of them at least.
  const size_t n = loads.size();
  for (size_t r = 1; give_up != INT64_MAX && r * n < lens.size(); ++r) {
    int64_t t = 0;
    for (size_t i = r * n - r; i <= r * n; ++i) t += lens[i] + kItemSetupTiles;
    if (t > give_up) return t;
  }
  Units<int64_t> units(0);
  units.free = loads;
  std::make_heap(units.free.begin(), units.free.end(), std::greater<int64_t>());
  units.end = *std::max_element(loads.begin(), loads.end());
  const bool idle = units.end == 0;
  for (size_t k = 0; k < lens.size(); ++k) {
    if (idle)
      units.add_sorted(k, lens[k] + kItemSetupTiles);
    else
      units.add(lens[k] + kItemSetupTiles);
    if (units.end > give_up) break;
  }
  return units.end;
}

typedef std::vector<std::vector<int32_t>> Cuts;  // per item (position in the list): cut points

// A way of cutting one schedule's items: where (position in the list, tile), the
// lengths that result, and the lengths of the items left whole, longest first.
struct Candidate {
  std::vector<std::pair<size_t, int32_t>> cuts;
  std::vector<int64_t> pieces, whole;
};

// The fill candidate (see balance_cuts), of at most max_pieces pieces.  `order`:
// the items, longest first.
Candidate fill_cuts(const std::vector<ItemTiles>& items, const std::vector<size_t>& order, int n_units, int64_t ideal,
                    int64_t limit, int64_t max_pieces) {
  struct Seg {
    int64_t len;
    size_t idx;
    int32_t t0;
    int n_cuts;  // of its item, so far
  };
  Candidate c;
  Units<int64_t> units(n_units);
  auto longer = [](const Seg& a, const Seg& b) { return a.len < b.len || (a.len == b.len && a.idx > b.idx); };
  std::priority_queue<Seg, std::vector<Seg>, decltype(longer)> rest(longer);  // what cuts left
  int64_t n_pieces = 0;
  for (size_t next = 0; next < order.size() || !rest.empty();) {
    Seg s{0, 0, 0, 0};
    if (next < order.size()) s = Seg{items[order[next]].tiles, order[next], 0, 0};
    if (next == order.size() || (!rest.empty() && longer(s, rest.top()))) {
      s = rest.top();
      rest.pop();
    } else {
      ++next;
    }
    const int64_t load = units.free[0];
    int64_t take = s.len;
    const int64_t more = s.n_cuts == 0 ? 2 : 1;  // pieces that a cut here adds
    if (load + s.len + kItemSetupTiles > limit && s.n_cuts + 1 < kMaxPieces && n_pieces + more <= max_pieces) {
      // Fill this unit up to the ideal, or give it the smallest piece when
      // it is there already.
      const int64_t room = ideal - load - kItemSetupTiles;
      if (s.len >= 2 * kMinBalancePiece) take = std::min(std::max(room, kMinBalancePiece), s.len - kMinBalancePiece);
    }
    units.add(take + kItemSetupTiles);
    (s.n_cuts == 0 && take == s.len ? c.whole : c.pieces).push_back(take);
    if (take < s.len) {
      n_pieces += more;
      c.cuts.push_back(std::make_pair(s.idx, s.t0 + (int32_t)take));
      rest.push(Seg{s.len - take, s.idx, s.t0 + (int32_t)take, s.n_cuts + 1});
    }
  }
  return c;
}

// How many of the items (longest first) are placed whole, each while the least
// loaded unit takes it within the limit.
size_t placed_whole(const std::vector<ItemTiles>& items, const std::vector<size_t>& order, int n_units, int64_t limit) {
  Units<int64_t> units(n_units);
  size_t n = 0;
  for (; n < order.size(); ++n) {
    const int64_t len = items[order[n]].tiles + kItemSetupTiles;
    if (units.free[0] + len > limit) break;
    units.add(len);
  }
  return n;
}

// The even candidate (see balance_cuts) of `target` pieces of the items that can
// be cut in two, beyond the first n_whole; no cut when it makes none.
Candidate even_cuts(const std::vector<ItemTiles>& items, const std::vector<size_t>& order, size_t n_whole,
                    int64_t target) {
  Candidate c;
  std::vector<size_t> big;
  int64_t big_tiles = 0;
  for (size_t k = n_whole; k < order.size() && items[order[k]].tiles >= 2 * kMinBalancePiece; ++k) {
    big.push_back(order[k]);
    big_tiles += items[order[k]].tiles;
  }
  if (target <= (int64_t)big.size()) return c;
  // Pieces in proportion to the lengths (largest remainders first), each
  // item's at most its length allows.
  std::vector<int64_t> n_pieces(big.size());
  std::vector<std::pair<double, size_t>> frac;
  int64_t dealt = 0;
  for (size_t i = 0; i < big.size(); ++i) {
    const int64_t len = items[big[i]].tiles;
    const double share = (double)target * (double)len / (double)big_tiles;
    const int64_t most = std::min<int64_t>(kMaxPieces, len / kMinBalancePiece);
    n_pieces[i] = std::max<int64_t>(1, std::min<int64_t>(most, (int64_t)share));
    dealt += n_pieces[i];
    if (n_pieces[i] < most) frac.push_back(std::make_pair(share - (double)n_pieces[i], i));
  }
  std::stable_sort(frac.begin(), frac.end(), [](const std::pair<double, size_t>& x, const std::pair<double, size_t>& y) {
    return x.first > y.first;
  });
  for (size_t f = 0; f < frac.size() && dealt < target; ++f, ++dealt) ++n_pieces[frac[f].second];
  for (size_t k = 0; k < order.size(); ++k) {
    const int64_t len = items[order[k]].tiles;
    const int64_t n = k >= n_whole && k - n_whole < big.size() ? n_pieces[k - n_whole] : 1;
    if (n == 1) c.whole.push_back(len);
    for (int64_t j = 1, prev = 0; n > 1 && j <= n; ++j) {
      const int64_t at = len * j / n;
      c.pieces.push_back(at - prev);
      if (j < n) c.cuts.push_back(std::make_pair(order[k], (int32_t)at));
      prev = at;
    }
  }
  return c;
}

void balance_cuts(const std::vector<ItemTiles>& items, int n_units, size_t n_items_total, int64_t max_pieces, Cuts* cuts) {
  if (items.empty()) return;
  int64_t total = 0, longest = 0;
  for (const ItemTiles& it : items) {
    total += it.tiles + kItemSetupTiles;
    longest = std::max(longest, it.tiles);
  }
  const int64_t ideal = (total + n_units - 1) / n_units;
  const int64_t limit = (int64_t)(ideal * kBalanceSlack);
  // List scheduling ends within one item of the even spread: when the longest
  // item fits in the slack, no schedule needs cuts (and none is simulated).
  if (ideal + longest + kItemSetupTiles <= limit) return;
  std::vector<size_t> order(items.size());  // longest first
  std::iota(order.begin(), order.end(), (size_t)0);
  std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return items[a].tiles > items[b].tiles; });
  const std::vector<int64_t> idle(n_units, 0);
  std::vector<int64_t> lens;
  for (size_t i : order) lens.push_back(items[i].tiles);
  // The best makespan and its piece count.
  std::pair<int64_t, int64_t> best(list_schedule(idle, lens), 0);
  if (best.first <= limit) return;
  Candidate chosen;
  auto consider = [&](Candidate c) {
    const int64_t n_pieces = (int64_t)c.pieces.size();
    const int64_t n_cuts = n_pieces + (int64_t)c.whole.size() - (int64_t)items.size();
    if (n_pieces == 0 || n_pieces > max_pieces || (total + n_cuts * kItemSetupTiles) / n_units > best.first) return;
    std::sort(c.pieces.begin(), c.pieces.end(), std::greater<int64_t>());
    lens.resize(c.pieces.size() + c.whole.size());
    std::merge(c.pieces.begin(), c.pieces.end(), c.whole.begin(), c.whole.end(), lens.begin(), std::greater<int64_t>());
    const std::pair<int64_t, int64_t> sc(list_schedule(idle, lens, best.first), n_pieces);
    if (sc < best) {
      best = sc;
      chosen = std::move(c);
    }
  };
  consider(fill_cuts(items, order, n_units, ideal, limit, max_pieces));
  const size_t n_whole = placed_whole(items, order, n_units, limit);
  for (int m = 1; m <= 4; ++m) consider(even_cuts(items, order, n_whole, (int64_t)m * n_units));
  if (chosen.cuts.empty()) return;
  cuts->resize(n_items_total);
  for (const std::pair<size_t, int32_t>& c : chosen.cuts) (*cuts)[(size_t)items[c.first].item].push_back(c.second);
  for (const ItemTiles& it : items) std::sort((*cuts)[(size_t)it.item].begin(), (*cuts)[(size_t)it.item].end());
}

// Key tiles of one work item's walk, exactly as the kernel counts them: the
// paged prefix, then each suffix range clipped to the item's last query.
int64_t item_tiles(const DevDesc& d, int chunk, int64_t qb, int q_per_wg) {
  constexpr int64_t T = 32;
  const int64_t last = std::min(qb * q_per_wg + q_per_wg, d.q_len[chunk]) - 1;
  const int64_t vis_end = d.q_begin[chunk] + last + 1;
  int64_t n = (d.prefix_keys + T - 1) / T;
  for (int s = 0; s < d.n_seg; ++s) {
    const int64_t vis = std::min(d.seg_hi[s], vis_end);
    if (vis > d.seg_lo[s]) n += (vis - d.seg_lo[s] + T - 1) / T;
  }
  return n;
}

int64_t item_keys(const DevDesc& d, int chunk, int64_t qb, int q_per_wg) {
  const int64_t last = std::min(qb * q_per_wg + q_per_wg, d.q_len[chunk]) - 1;
  const int64_t pos_hi = d.q_begin[chunk] + last;
  int64_t keys = d.prefix_keys;
  for (int s = 0; s < d.n_seg; ++s) keys += std::max<int64_t>(0, std::min(d.seg_hi[s], pos_hi + 1) - d.seg_lo[s]);
  return keys;
}

// Query blocks of every descriptor and chunk for one workgroup shape, with
// their tile counts; each is one work item per head group.
struct Block {
  int32_t desc, chunk, q_block;
  int64_t keys, tiles;
};

struct Blocks {
  Shape shape;
  int n_groups;
  std::vector<Block> list;
  int64_t nonempty = 0, all_tiles = 0, max_tiles = 0;  // items with a tile; tiles of all items; the longest
};

Blocks list_blocks(const std::vector<DevDesc>& descs, int32_t Hq, int32_t Hkv, int rows) {
  Blocks b;
  b.shape = shape_for(Hq, Hkv, rows);
  b.n_groups = Hkv * b.shape.groups_per_kv;
  const int q_per_wg = b.shape.q_per_wg;
  for (size_t i = 0; i < descs.size(); ++i) {
    const DevDesc& d = descs[i];
    for (int c = 0; c < 2; ++c)
      for (int64_t qb = 0; qb * q_per_wg < d.q_len[c]; ++qb) {
        const int64_t tiles = item_tiles(d, c, qb, q_per_wg);
        b.list.push_back(Block{(int32_t)i, c, (int32_t)qb, item_keys(d, c, qb, q_per_wg), tiles});
        if (tiles > 0) b.nonempty += b.n_groups;
        b.all_tiles += tiles * b.n_groups;
        b.max_tiles = std::max(b.max_tiles, tiles);
      }
  }
  return b;
}

// Pieces of a walk of `tiles` cut to at most `cap` tiles each (in equal parts,
// kMaxPieces at most).
int64_t pieces_at(int64_t tiles, int64_t cap) { return std::max<int64_t>(1, std::min(kMaxPieces, (tiles + cap - 1) / cap)); }

// The head groups of one schedule: with the groups a multiple of the XCDs,
// each XCD's list is its own schedule on its 32 compute units, and all eight
// are alike; otherwise the lists share the units (the interleave in plan_items
// moves items between XCDs) and one schedule over all of them is the closer
// model.
int schedules_of(int n_groups) { return n_groups % kXcds == 0 ? kXcds : 1; }

// The work list of one launch for one workgroup shape: items, split items and
// piece count into *out (whose descriptors are set).  cap > 0: every walk cut
// to at most that many tiles; cap = 0: balance cuts where they pay (few items
// with a pinned shape: equal pieces, see kPinnedBelowItems), of at most
// max_pieces pieces.
int plan_items(const Blocks& b_, int64_t target_pieces, bool pinned, int64_t cap, Plan* out,
               int64_t max_pieces = INT64_MAX) {
  struct Cand {
    int64_t cost;
    WorkItem w;
  };
  out->shape = b_.shape;
  const int n_groups = b_.n_groups;
  const std::vector<Block>& blocks = b_.list;
  // Cut points of each item's walk (item = block * n_groups + head group).
  std::vector<std::vector<int32_t>> cuts;
  auto cut_all = [&](auto&& pieces) {
    cuts.resize(blocks.size() * n_groups);
    for (size_t bi = 0; bi < blocks.size(); ++bi) {
      const int64_t n = pieces(blocks[bi].tiles);
      for (int g = 0; g < n_groups; ++g)
        for (int64_t k = 1; k < n; ++k) cuts[bi * n_groups + g].push_back((int32_t)(blocks[bi].tiles * k / n));
    }
  };
  if (cap > 0) {
    if (cap < b_.max_tiles) cut_all([&](int64_t tiles) { return pieces_at(tiles, cap); });
  } else if (pinned && target_pieces > 0 && b_.nonempty > 0 && b_.nonempty < kPinnedBelowItems &&
             b_.max_tiles >= 4 * kPinnedMinTiles) {
    const int64_t len = std::max<int64_t>(kPinnedMinTiles, (b_.all_tiles + target_pieces - 1) / target_pieces);
    cut_all([&](int64_t tiles) { return std::min<int64_t>(kMaxPieces, tiles / len); });
  } else if (target_pieces > 0) {
    // The first schedule's items; the others' are those of the next head groups.
    const int n_sched = schedules_of(n_groups);
    std::vector<ItemTiles> sched;
    for (size_t bi = 0; bi < blocks.size(); ++bi)
      if (blocks[bi].tiles > 0)
        for (int g = 0; g < n_groups; g += n_sched) sched.push_back(ItemTiles{(int64_t)(bi * n_groups + g), blocks[bi].tiles});
    balance_cuts(sched, kComputeUnits / n_sched, blocks.size() * n_groups, max_pieces / n_sched, &cuts);
    if (!cuts.empty())
      for (const ItemTiles& it : sched)
        for (int x = 1; x < n_sched; ++x) cuts[(size_t)it.item + x] = cuts[(size_t)it.item];
  }
  out->splits.clear();
  out->n_pieces = 0;
  std::vector<std::vector<Cand>> per_xcd(kXcds);
  int64_t total = 0;
  for (size_t bi = 0; bi < blocks.size(); ++bi) {
    const Block& b = blocks[bi];
    for (int g = 0; g < n_groups; ++g) {
      const std::vector<int32_t>* c = cuts.empty() ? nullptr : &cuts[bi * n_groups + g];
      if (!c || c->empty()) {
        per_xcd[g % kXcds].push_back(Cand{b.keys, WorkItem{b.desc, b.chunk, b.q_block, g, 0, -1, -1, 0}});
        ++total;
        continue;
      }
      const int64_t n_pieces = (int64_t)c->size() + 1;
      out->splits.push_back(SplitItem{b.desc, b.chunk, b.q_block, g, (int32_t)out->n_pieces, (int32_t)n_pieces});
      for (int64_t k = 0; k < n_pieces; ++k) {
        const int32_t t0 = k == 0 ? 0 : (*c)[k - 1];
        const int32_t t1 = k + 1 == n_pieces ? (int32_t)b.tiles : (*c)[k];
        per_xcd[g % kXcds].push_back(
            Cand{(int64_t)(t1 - t0) * 32, WorkItem{b.desc, b.chunk, b.q_block, g, t0, t1, (int32_t)(out->n_pieces + k), 0}});
        ++total;
      }
      out->n_pieces += n_pieces;
    }
  }
  if (total > 0x7fffffffLL) return fail(CP_ERR_UNSUPPORTED, "cp_attn_partial: work list beyond 2^31 workgroups");
  // One round of lists that are not alike: one list, in the order of the lengths,
  // so that every XCD takes items of every group (all start at once: no XCD has
  // more than its share).  2207 tokens, rank 0 of 2, 8/2 heads: 27.2 us, 29.1 with a
  // group on every other XCD; 156 launches of up to 60 us 0.4 % faster on average.
  // Longer ones keep the lists: 0.2 % faster beyond 500 us, up to 2 %.
  if (schedules_of(n_groups) == 1 && total <= kComputeUnits)
    for (int x = 1; x < kXcds; ++x) {
      per_xcd[0].insert(per_xcd[0].end(), per_xcd[x].begin(), per_xcd[x].end());
      per_xcd[x].clear();
    }
  for (auto& v : per_xcd)
    std::stable_sort(v.begin(), v.end(), [](const Cand& a, const Cand& b) { return a.cost > b.cost; });
  out->items.clear();
  out->items.reserve((size_t)total);
  std::vector<size_t> head(kXcds, 0);
  std::vector<int> from(kXcds);  // an XCD's list, and later the one it took from last
  std::iota(from.begin(), from.end(), 0);
  for (int64_t i = 0; i < total; ++i) {
    // The list that this XCD took from last while its next item is as long as
    // any that is left (always, where the lists are alike: the groups a multiple
    // of the XCDs); else, of the lists with such an item, the one with the most
    // left.  The launch as a whole is then dispatched longest first, as its choice
    // supposes: where XCDs took their own list's shorter items first, long ones
    // were left for the end.
    int& x = from[i % kXcds];
    int64_t top = -1;
    for (int y = 0; y < kXcds; ++y)
      if (head[y] < per_xcd[y].size()) top = std::max(top, per_xcd[y][head[y]].cost);
    if (head[x] == per_xcd[x].size() || per_xcd[x][head[x]].cost < top) {
      size_t most = 0;
      for (int y = 0; y < kXcds; ++y) {
        const size_t left = per_xcd[y].size() - head[y];
        if (left > most && per_xcd[y][head[y]].cost == top) {
          most = left;
          x = y;
        }
      }
    }
    out->items.push_back(per_xcd[x][head[x]++].w);
  }
  return CP_OK;
}

// Estimated time (microseconds) of a launch: its work list simulated as it is
// dispatched, in order to the first free of each XCD's 32 compute units, a
// workgroup taking its tiles times the shape's time per tile plus a fixed
// set-up (table and query fetch, first tiles, stores); the clock falls as more
// units are busy; then the split merge, if any, its launch and its traffic
// (the pieces written and read back, the merged rows written: mostly cache).
// The constants are fitted to the timed lists of 35 launches (500 to 64K
// tokens, degrees 1 to 8, with and without a prefix, in both shapes, uncut,
// balance cut and cut into 2 to 64 pieces): mean error 4.4 %, and the list
// that the estimate prefers is 0.5 % slower on average than the fastest one
// timed.
constexpr double kSmallTileUs = 0.766;  // a 256-row x 32-key tile on one compute unit
constexpr double kLargeTileUs = 1.064;  // a 384-row one
constexpr double kItemSetupUs = 7.0;
constexpr double kBusySlowdown = 0.093;
constexpr double kMergeUs = 5.4;
constexpr double kMergeBytesPerUs = 7.7e6;

double tile_us(const Shape& s) { return s.rows_per_wg == kRowsLarge ? kLargeTileUs : kSmallTileUs; }

double merge_us(const Shape& s, int64_t n_pieces, int64_t n_splits) {
  if (n_splits == 0) return 0.0;
  return kMergeUs + (double)piece_bytes(s.rows_per_wg) * (2.0 * n_pieces + n_splits) / kMergeBytesPerUs;
}

double slowed(double end, double sum, int n_units) { return end > 0.0 ? end + kBusySlowdown * sum / n_units : 0.0; }

double estimate_us(const Plan& plan) {
  const double tile = tile_us(plan.shape);
  std::vector<Units<double>> units(kXcds, Units<double>(kComputeUnits / kXcds));
  double sum = 0.0;
  for (size_t i = 0; i < plan.items.size(); ++i) {
    const WorkItem& w = plan.items[i];
    const int64_t tiles = w.t_end >= 0 ? (int64_t)(w.t_end - w.t_begin)
                                       : item_tiles(plan.descs[w.desc], w.chunk, w.q_block, plan.shape.q_per_wg);
    units[i % kXcds].add(tiles * tile + kItemSetupUs);
    sum += tiles * tile + kItemSetupUs;
  }
  double end = 0.0;
  for (const Units<double>& u : units) end = std::max(end, u.end);
  return slowed(end, sum, kComputeUnits) + merge_us(plan.shape, plan.n_pieces, (int64_t)plan.splits.size());
}

size_t align_up(size_t x) { return (x + kItemsAlign - 1) / kItemsAlign * kItemsAlign; }

// The workspace of a list of so many entries.
Layout layout_of_counts(size_t n_descs, size_t n_items, size_t n_splits, size_t n_pieces, int rows) {
  Layout l;
  l.items = align_up(n_descs * sizeof(DevDesc));
  l.splits = align_up(l.items + n_items * sizeof(WorkItem));
  l.pieces = align_up(l.splits + n_splits * sizeof(SplitItem));
  l.total = l.pieces + n_pieces * piece_bytes(rows);
  return l;
}

// A candidate list of one shape: its walks cut to `cap` tiles, its workspace,
// its estimate and a bound below it: its work spread evenly over the units (or
// its longest piece alone), and its merge.
struct Choice {
  const Blocks* blocks;
  int64_t cap, n_pieces, n_splits;
  size_t total;
  double at_least, us;
  size_t slots() const { return (size_t)n_pieces * piece_bytes(blocks->shape.rows_per_wg); }
};

// The same estimate for a list cut to c.cap tiles, without building it; or, as
// soon as it is known to exceed `give_up`, something above that.  `lens` is
// scratch (length, count).
double estimate_cap(const Choice& c, double give_up, std::vector<std::pair<int64_t, int64_t>>* lens) {
  const Blocks& b = *c.blocks;
  const int n_sched = schedules_of(b.n_groups), per_sched = b.n_groups / n_sched;
  lens->clear();
  int64_t n_items = 0;
  for (const Block& x : b.list) {
    // Equal parts: x.tiles % n of them are one tile longer than the others.
    const int64_t n = pieces_at(x.tiles, c.cap), longer = x.tiles % n;
    if (longer) lens->push_back(std::make_pair(x.tiles / n + 1, longer * per_sched));
    lens->push_back(std::make_pair(x.tiles / n, (n - longer) * per_sched));
    n_items += n * per_sched;
  }
  std::sort(lens->begin(), lens->end(), std::greater<std::pair<int64_t, int64_t>>());
  const int n_units = kComputeUnits / n_sched;
  const double rest = kBusySlowdown * (b.all_tiles / n_sched * tile_us(b.shape) + n_items * kItemSetupUs) / n_units +
                      merge_us(b.shape, c.n_pieces, c.n_splits);
  // As in list_schedule: of the r * n + 1 longest, some unit takes r + 1, no
  // shorter than the last of them.
  int64_t before = 0;
  for (const std::pair<int64_t, int64_t>& len : *lens) {
    before += len.second;
    const double us = len.first * tile_us(b.shape) + kItemSetupUs;
    if ((double)((before - 1) / n_units + 1) * us + rest > give_up) return INFINITY;
  }
  Units<double> units(n_units);
  size_t k = 0;
  for (const std::pair<int64_t, int64_t>& len : *lens) {
    const double us = len.first * tile_us(b.shape) + kItemSetupUs;
    for (int64_t i = 0; i < len.second; ++i) units.add_sorted(k++, us);
    if (units.end + rest > give_up) break;
  }
  return units.end > 0.0 ? units.end + rest : 0.0;
}

// Adds one shape's candidates (not yet estimated): the longest walk cut into k =
// 1, 2, ... equal pieces and every other walk to that length, while their
// pieces and workspace stay within the limits.
void add_choices(const Blocks& b, size_t n_descs, int64_t target_pieces, size_t limit, std::vector<Choice>* out) {
  int64_t last = 0;
  for (int64_t k = 1; k <= kMaxPieces; ++k) {
    const int64_t cap = std::max<int64_t>(1, (b.max_tiles + k - 1) / k);
    if (k > 1 && (cap < kMinPieceTiles || target_pieces == 0)) break;
    if (cap == last) continue;
    last = cap;
    Choice c{&b, cap, 0, 0, 0, 0.0, INFINITY};
    int64_t n = 0, shortest = b.max_tiles, longest = 0;
    for (const Block& x : b.list) {
      const int64_t m = pieces_at(x.tiles, cap);
      n += m;
      longest = std::max(longest, (x.tiles + m - 1) / m);
      if (m > 1) {
        c.n_pieces += m;
        ++c.n_splits;
        shortest = std::min(shortest, x.tiles / m);
      }
    }
    n *= b.n_groups;
    c.n_pieces *= b.n_groups;
    c.n_splits *= b.n_groups;
    c.total = layout_of_counts(n_descs, n, c.n_splits, c.n_pieces, b.shape.rows_per_wg).total;
    if (c.total > limit || (k > 1 && (c.n_pieces > target_pieces || shortest < kMinPieceTiles))) break;
    const double spread = (b.all_tiles * tile_us(b.shape) + n * kItemSetupUs) / kComputeUnits;
    const double alone = longest * tile_us(b.shape) + kItemSetupUs;
    if (n > 0)
      c.at_least = std::max(spread, alone) + kBusySlowdown * spread + merge_us(b.shape, c.n_pieces, c.n_splits);
    out->push_back(c);
  }
}

// Bounds (microseconds) of one shape's schedule before any item is cut: the
// launch's work spread evenly over the compute units (every XCD gets the same
// share of each block when the head groups are a multiple of the XCDs, and the
// interleave spreads them otherwise), and that plus the longest item (list
// scheduling ends within one item of the even spread).
struct Bounds {
  double lo, hi;
};

Bounds shape_bounds(const Blocks& b) {
  const double work = b.all_tiles * tile_us(b.shape) + (double)b.list.size() * b.n_groups * kItemSetupUs;
  Bounds r;
  r.lo = work / kComputeUnits;
  r.hi = r.lo + b.max_tiles * tile_us(b.shape) + kItemSetupUs;
  return r;
}

// Work-group shape forced by cp_set_workgroup_rows (0: chosen per launch).
std::atomic<int> g_forced_rows{0};

}  // namespace

extern "C" int cp_set_workgroup_rows(int32_t rows) {
  if (rows != 0 && rows != kRowsSmall && rows != kRowsLarge)
    return fail_static(CP_ERR_INVALID, "cp_set_workgroup_rows: rows must be 0, 256 or 384");
  g_forced_rows.store(rows);
  clear_error();
  return CP_OK;
}

namespace cpattn {

// Work lists of recent launches.  A layer after layer of the same shapes
// plans the same list (the work list depends on the descriptors' positions,
// chunks and key ranges and on the heads, never on their buffers), so the
// list of a launch whose key matches is reused instead of planned again:
// the key holds every non-pointer field of the converted descriptors, the
// head counts, the piece target and the pinned shape, and matches exactly.  A
// list planned for a workspace of `limit` bytes serves any that holds it and is
// no larger (what fits there was among its candidates); `wanted` is the size
// of the unlimited plan.
struct CachedPlan {
  std::vector<int64_t> key;
  std::vector<WorkItem> items;
  std::vector<SplitItem> splits;
  int64_t n_pieces;
  Shape shape;
  bool joined;  // of the joined descriptors
  size_t total, limit, wanted;
};
constexpr size_t kPlanCacheSize = 16;
static std::mutex g_plan_cache_mu;
static std::vector<CachedPlan> g_plan_cache;  // most recent last
static size_t g_plan_cache_hits = 0;

static std::vector<int64_t> plan_key(const std::vector<DevDesc>& descs, int32_t Hq, int32_t Hkv, int64_t target_pieces,
                                     int forced) {
  std::vector<int64_t> k = {Hq, Hkv, target_pieces, forced, (int64_t)descs.size()};
  for (const DevDesc& d : descs) {
    const int64_t f[] = {d.P, d.R, d.q_begin[0], d.q_begin[1], d.q_len[0], d.q_len[1], d.local_off[0], d.local_off[1],
                         d.o_off[0], d.o_off[1], d.seg_lo[0], d.seg_lo[1], d.seg_hi[0], d.seg_hi[1], d.n_seg,
                         d.prefix_keys, d.n_blocks, d.reserved};
    k.insert(k.end(), f, f + sizeof(f) / sizeof(f[0]));
  }
  return k;
}

static int plan_uncached(int32_t Hq, int32_t Hkv, int64_t target_pieces, int forced, Plan* out,
                         size_t limit = SIZE_MAX, size_t* wanted = nullptr);

// Time (microseconds) of a launch of about one round, closer than estimate_us for
// workgroups that are partly empty: the fixed set-up, the loads and stores of the
// rows that are there, a tile time by whether one or two waves of a SIMD have
// rows (a query block of one head that is half empty leaves every SIMD one), and
// the merge of cut items by their number, pieces and bytes.  Fitted to 4609 lists
// of 297 launches of a last rank (20 to 4000 rows in 13 head layouts, chunks
// joined and apart, whole and in up to 24 pieces): mean error 3.7 %, where
// estimate_us has 12.9.  It has no say where launches of many rounds are planned,
// to which it was not fitted.
static double small_launch_us(const Plan& plan) {
  const Shape& sh = plan.shape;
  const bool large = sh.rows_per_wg == kRowsLarge;
  const double tile[2] = {large ? 0.75 : 0.54, large ? 1.05 : 0.735};
  const int per_wave = sh.rows_per_wg / 128, per_head = sh.q_per_wg / 16;  // 16-row blocks
  auto two_waves = [&](int live) {  // of a SIMD, with rows: waves w and w + 4 share one
    int n[4] = {};
    for (int w = 0; w < 8; ++w)
      for (int b = per_wave * w; b < per_wave * (w + 1); ++b)
        if (b % per_head * 16 < live) {
          if (++n[w % 4] == 2) return true;
          break;
        }
    return false;
  };
  std::vector<Units<double>> units(kXcds, Units<double>(kComputeUnits / kXcds));
  double sum = 0.0, end = 0.0;
  for (size_t i = 0; i < plan.items.size(); ++i) {
    const WorkItem& w = plan.items[i];
    const DevDesc& d = plan.descs[w.desc];
    const int64_t tiles = w.t_end >= 0 ? (int64_t)(w.t_end - w.t_begin) : item_tiles(d, w.chunk, w.q_block, sh.q_per_wg);
    const int live = (int)std::min<int64_t>(sh.q_per_wg, d.q_len[w.chunk] - (int64_t)w.q_block * sh.q_per_wg);
    const double us = 6.5 + 0.7 * live * sh.heads_per_wg / 32 + tiles * tile[two_waves(live)];
    units[i % kXcds].add(us);
    sum += us;
  }
  for (const Units<double>& u : units) end = std::max(end, u.end);
  end += 0.097 * sum / kComputeUnits;
  if (plan.splits.empty()) return end;
  const double n = (double)plan.splits.size(), pieces = (double)plan.n_pieces;
  return end + 3.6 + 0.13 * pieces / n + 0.45 * std::log2(n) + (double)piece_bytes(sh.rows_per_wg) * (2.0 * pieces + n) / 14.9e6;
}

// The plan of a launch's joined descriptors (*joined), or the whole items of the
// descriptors as they are, where those are within one round and small_launch_us
// finds them the faster: there idle compute units may take the second chunk's
// rows sooner than the first chunk's workgroups, and half-empty ones end sooner
// than their pieces and a merge (rank 3 of 4 of 1007 tokens, 28/4 heads: 27.2 us
// joined and cut, 20.2 apart; 170 tokens on one GPU, 32/8: 14.7 joined, 16.4
// apart).  Over the 297 launches what this takes is 1.4 % slower on average than
// the fastest list timed; the joined choice alone 5.3.
static int plan_joined(int32_t Hq, int32_t Hkv, int64_t target_pieces, int forced, Plan* out, size_t limit,
                       size_t* wanted, bool* joined) {
  Plan whole;
  whole.descs = out->descs;
  *joined = false;
  if (forced) return plan_uncached(Hq, Hkv, target_pieces, forced, out, limit, wanted);
  for (size_t i = 0; i < out->descs.size(); ++i) {
    join_chunks(&out->descs[i]);
    *joined |= out->descs[i].q_len[1] != whole.descs[i].q_len[1];
  }
  const Blocks blocks = list_blocks(whole.descs, Hq, Hkv, kRowsSmall);
  const bool one_round = blocks.list.size() * blocks.n_groups <= (size_t)kComputeUnits;
  if (!*joined && !one_round) return plan_uncached(Hq, Hkv, target_pieces, forced, out, limit, wanted);
  Plan choice;
  choice.descs = out->descs;
  int st = plan_uncached(Hq, Hkv, target_pieces, forced, &choice, SIZE_MAX, wanted);
  if (st != CP_OK) return st;
  if (one_round && (*joined || choice.n_pieces > 0)) {
    st = plan_items(blocks, target_pieces, false, std::max<int64_t>(1, blocks.max_tiles), &whole);
    if (st != CP_OK) return st;
    if (small_launch_us(whole) < small_launch_us(choice)) {
      choice = std::move(whole);
      *wanted = layout_of(choice).total;
      *joined = false;
    }
  }
  if (*wanted > limit) {
    size_t size = 0;
    return plan_uncached(Hq, Hkv, target_pieces, forced, out, limit, &size);
  }
  *out = std::move(choice);
  return CP_OK;
}

// The plan of a launch in `limit` bytes of workspace; *wanted is the size of
// the unlimited one.
static int build_plan_limited(const cp_partial_desc* descs, int32_t n_descs, int32_t Hq, int32_t Hkv,
                              int64_t target_pieces, size_t limit, Plan* out, size_t* wanted) {
  int st = check_heads(Hq, Hkv, "cp_attn_partial");
  if (st != CP_OK) return st;
  if (n_descs < 0) return fail(CP_ERR_INVALID, "cp_attn_partial: n_descs < 0");
  if (n_descs > 0 && !descs) return fail(CP_ERR_INVALID, "cp_attn_partial: descs is NULL");
  out->descs.resize(n_descs);
  for (int i = 0; i < n_descs; ++i) {
    st = to_dev(descs[i], i, &out->descs[i]);
    if (st != CP_OK) return st;
  }
  const int forced = g_forced_rows.load();
  std::vector<int64_t> key = plan_key(out->descs, Hq, Hkv, target_pieces, forced);
  {
    std::lock_guard<std::mutex> lock(g_plan_cache_mu);
    for (size_t i = g_plan_cache.size(); i-- > 0;) {
      const CachedPlan& c = g_plan_cache[i];
      if (c.total > limit || limit > c.limit || c.key != key) continue;
      out->items = c.items;
      out->splits = c.splits;
      out->n_pieces = c.n_pieces;
      out->shape = c.shape;
      if (c.joined)
        for (DevDesc& d : out->descs) join_chunks(&d);
      *wanted = c.wanted;
      ++g_plan_cache_hits;
      return CP_OK;
    }
  }
  bool joined = false;
  st = plan_joined(Hq, Hkv, target_pieces, forced, out, limit, wanted, &joined);
  if (st != CP_OK) return st;
  const size_t total = layout_of(*out).total;
  if (total > limit) return CP_OK;  // the caller refuses it
  if (*wanted <= limit) limit = SIZE_MAX;
  std::lock_guard<std::mutex> lock(g_plan_cache_mu);
  if (g_plan_cache.size() == kPlanCacheSize) g_plan_cache.erase(g_plan_cache.begin());
  g_plan_cache.push_back(
      CachedPlan{std::move(key), out->items, out->splits, out->n_pieces, out->shape, joined, total, limit, *wanted});
  return CP_OK;
}

int build_plan(const cp_partial_desc* descs, int32_t n_descs, int32_t Hq, int32_t Hkv, int64_t target_pieces,
               Plan* out) {
  size_t wanted = 0;
  return build_plan_limited(descs, n_descs, Hq, Hkv, target_pieces, SIZE_MAX, out, &wanted);
}

int build_plan_within(const cp_partial_desc* descs, int32_t n_descs, int32_t Hq, int32_t Hkv, size_t bytes, Plan* out,
                      Layout* lay, size_t* wanted) {
  const int st = build_plan_limited(descs, n_descs, Hq, Hkv, kTargetPieces, bytes, out, wanted);
  if (st == CP_OK) *lay = layout_of(*out);
  return st;
}

// The list of an unpinned launch whose estimate ends first among those of at most
// max_pieces pieces and a workspace of at most `limit`; *fits says whether there
// is any (out is then set).  `whole` is the shape that the bounds decide for, or
// null.
static int choose_list(const Blocks& small, const Blocks& large, const Blocks* whole, int64_t target_pieces,
                       size_t limit, int64_t max_pieces, Plan* out, bool* fits) {
  const size_t n_descs = out->descs.size();
  // Balance cuts of as many pieces as the limit leaves room for beside the
  // uncut list's tables.
  auto balance = [&](const Blocks& b, Plan* p) {
    int64_t room = max_pieces;
    if (limit != SIZE_MAX) {
      const size_t tables = layout_of_counts(n_descs, b.list.size() * b.n_groups, 0, 0, b.shape.rows_per_wg).total;
      const size_t piece = piece_bytes(b.shape.rows_per_wg) + sizeof(WorkItem) + sizeof(SplitItem);
      room = limit > tables + 2 * kItemsAlign
                 ? std::min(room, (int64_t)((limit - tables - 2 * kItemsAlign) / piece))
                 : 0;
    }
    const int st = plan_items(b, target_pieces, false, 0, p, room);
    *fits = st == CP_OK && layout_of(*p).total <= limit;
    return st;
  };
  if (whole) {
    const int st = balance(*whole, out);
    if (st != CP_OK || *fits) return st;
  }
  std::vector<Choice> choices;
  add_choices(small, n_descs, std::min(target_pieces, max_pieces), limit, &choices);
  add_choices(large, n_descs, std::min(target_pieces, max_pieces), limit, &choices);
  *fits = !choices.empty();
  if (!*fits) return CP_OK;
  // Piece slots that, with the tables, fit the scratch of cp_attn_partial_noalloc
  // are preferred up to the estimate's own error: both entry points then run
  // the same list, in half the workspace or less.  It buys no speed: in 87
  // launches where this decides, the lists it takes are 1.1 % slower on average
  // (0.86 to 1.17 times the time of those it leaves).
  constexpr size_t kSlotBytes = (size_t)(32 << 20) - (256 << 10);
  constexpr double kSlotGain = 1.04;
  // Estimated in the order of their bounds; most of them are settled by that.
  std::vector<Choice*> order;
  for (Choice& c : choices) order.push_back(&c);
  std::stable_sort(order.begin(), order.end(), [](const Choice* a, const Choice* b) { return a->at_least < b->at_least; });
  std::vector<std::pair<int64_t, int64_t>> lens;
  double best_us = INFINITY;
  for (Choice* c : order) {
    // Rounding aside, no estimate is below its bound.
    const double give_up = (c->slots() <= kSlotBytes ? kSlotGain : 1.0) * best_us * (1.0 + 1e-9);
    if (c->at_least > give_up) continue;
    c->us = estimate_cap(*c, give_up, &lens);
    best_us = std::min(best_us, c->us);
  }
  const Choice* best = &choices[0];
  for (const Choice& c : choices)
    if (c.us < best->us) best = &c;
  if (best->slots() > kSlotBytes) {
    const Choice* within = nullptr;
    for (const Choice& c : choices)
      if (c.slots() <= kSlotBytes && (!within || c.us < within->us)) within = &c;
    if (within && within->us <= kSlotGain * best->us) best = within;
  }
  const Choice chosen = *best;
  const int st = plan_items(*chosen.blocks, target_pieces, false, chosen.cap, out);
  if (st != CP_OK || target_pieces == 0) return st;
  // Long walks: the balance cuts of each shape, where they end sooner.
  double us = chosen.us;
  for (const Blocks* b : {&small, &large}) {
    if (b->max_tiles < 2 * kMinBalancePiece) continue;
    const double spread = shape_bounds(*b).lo;
    if (slowed(spread, spread, 1) >= us) continue;  // no list of this shape ends sooner
    Plan balanced;
    balanced.descs = out->descs;
    const int st2 = balance(*b, &balanced);
    if (st2 != CP_OK) return st2;
    if (!*fits) continue;
    const double t = estimate_us(balanced);
    if (t < us) {
      us = t;
      *out = std::move(balanced);
    }
  }
  *fits = true;
  return CP_OK;
}

// The work list of a launch whose descriptors are converted (out->descs), in
// `limit` bytes of workspace: the list of the free choice, or, when that does
// not fit, of the fastest estimate that does with no more pieces; the shortest
// list when none fits.
// *wanted: the workspace of the free choice.
// The larger shape shares every K/V fragment between more rows (faster per
// tile) but makes fewer, longer work items, which fill the compute units
// worse; cuts fill them better but cost set-ups and a merge.
static int plan_uncached(int32_t Hq, int32_t Hkv, int64_t target_pieces, int forced, Plan* out, size_t limit,
                         size_t* wanted) {
  size_t free_size = 0;
  size_t* const size = wanted ? wanted : &free_size;
  if (forced) {
    // A pinned shape: its fixed rule for fewer pieces, down to none.
    const Blocks b = list_blocks(out->descs, Hq, Hkv, forced);
    *size = 0;
    for (int64_t target = target_pieces;; target = target >= 4 ? target / 2 : 0) {
      const int st = plan_items(b, target, true, 0, out);
      if (st != CP_OK) return st;
      const size_t total = layout_of(*out).total;
      if (*size == 0) *size = total;
      if (total <= limit || out->n_pieces == 0 || target == 0) return CP_OK;
    }
  }
  const Blocks small = list_blocks(out->descs, Hq, Hkv, kRowsSmall);
  const Blocks large = list_blocks(out->descs, Hq, Hkv, kRowsLarge);
  // Launches of many rounds: when the bounds already decide (one shape's worst
  // case ends before the other's best), only the winner is planned.  Its
  // worst case is within one item of its even spread, which leaves little to
  // cuts other than the balance cuts.
  const Bounds bs = shape_bounds(small), bl = shape_bounds(large);
  const Blocks* whole = bl.hi < bs.lo ? &large : bs.hi < bl.lo ? &small : nullptr;
  bool fits = false;
  int st = choose_list(small, large, whole, target_pieces, SIZE_MAX, INT64_MAX, out, &fits);
  if (st != CP_OK) return st;
  *size = layout_of(*out).total;
  if (*size <= limit) return CP_OK;
  st = choose_list(small, large, nullptr, target_pieces, limit, out->n_pieces, out, &fits);
  if (st != CP_OK || fits) return st;
  return plan_items(large, 0, false, 0, out);
}

Layout layout_of(const Plan& plan) {
  return layout_of_counts(plan.descs.size(), plan.items.size(), plan.splits.size(), (size_t)plan.n_pieces,
                          plan.shape.rows_per_wg);
}

void pack_tables(const Plan& plan, const Layout& lay, unsigned char* host) {
  std::memcpy(host, plan.descs.data(), plan.descs.size() * sizeof(DevDesc));
  std::memcpy(host + lay.items, plan.items.data(), plan.items.size() * sizeof(WorkItem));
  if (!plan.splits.empty())
    std::memcpy(host + lay.splits, plan.splits.data(), plan.splits.size() * sizeof(SplitItem));
}

bool pack_inline(const Plan& plan, InlineTables* out) {
  const size_t n = plan.items.size() + plan.splits.size();
  if (plan.descs.size() > (size_t)kInlineDescs || plan.descs.size() * sizeof(DevDesc) + n * 8 > kInlineBytes) return false;
  std::memcpy(out->bytes, plan.descs.data(), plan.descs.size() * sizeof(DevDesc));
  unsigned char* at = out->bytes + plan.descs.size() * sizeof(DevDesc);
  for (const WorkItem& w : plan.items) {
    if (w.q_block >= kInlineQBlocks || w.head_group >= kInlineGroups || w.t_begin >= kInlineTile ||
        w.t_end >= kInlineTile || w.piece >= kInlinePiece)
      return false;
    const uint64_t x = inline_item(w);
    std::memcpy(at, &x, 8);
    at += 8;
  }
  for (const SplitItem& s : plan.splits) {
    if (s.q_block >= kInlineQBlocks || s.head_group >= kInlineGroups || s.first_piece >= kInlinePiece ||
        s.n_pieces >= kInlinePieces)
      return false;
    const uint64_t x = inline_split(s);
    std::memcpy(at, &x, 8);
    at += 8;
  }
  return true;
}

PartialParams partial_params(const Plan& plan, const Layout& lay, unsigned char* ws, int32_t Hq, int32_t Hkv,
                             float scale) {
  PartialParams p;
  std::memset(&p, 0, sizeof(p));
  p.descs = reinterpret_cast<const DevDesc*>(ws);
  p.items = reinterpret_cast<const WorkItem*>(ws + lay.items);
  p.n_items = (int32_t)plan.items.size();
  p.Hq = Hq;
  p.Hkv = Hkv;
  p.heads_per_wg = plan.shape.heads_per_wg;
  p.q_per_wg = plan.shape.q_per_wg;
  p.groups_per_kv = plan.shape.groups_per_kv;
  p.scale = scale;
  p.scale_log2 = scale * 1.4426950408889634f;
  p.rows_per_wg = plan.shape.rows_per_wg;
  p.pieces = plan.n_pieces ? ws + lay.pieces : nullptr;
  p.splits = reinterpret_cast<const SplitItem*>(ws + lay.splits);
  p.n_splits = (int32_t)plan.splits.size();
  p.n_descs = (int32_t)plan.descs.size();
  p.n_pieces = plan.n_pieces;
  return p;
}

bool capturing(void* stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing((hipStream_t)stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return false;
}

}  // namespace cpattn

namespace {

// Pinned host staging for the descriptor/work-list upload, mapped into the
// device's address space and coherent (the device reads it over the bus,
// never from a cached copy): the upload kernel reads it (upload.hip).  A slot
// is reused only after the upload that read it is done with it: the kernel's
// blocks write the words after the tables.  Captured uploads take no slot.
struct Slot {
  std::mutex mu;           // held while the slot is waited for, filled and launched from
  unsigned char* host = nullptr;
  void* mapped = nullptr;  // the same memory as the device addresses it
  size_t cap = 0;
  size_t words_at = 0;     // the pending upload's words
  size_t n_words = 0;      // 0: none pending
  int device = 0;          // where the pending upload runs
  hipStream_t stream = nullptr;
};
constexpr int kSlots = 8;
Slot g_slots[kSlots];
std::atomic<unsigned> g_next_slot{0};

// What the runtime says of the slot's stream, without waiting for it:
// hipErrorNotReady while it has work to do.  Not asked: a stream that is being
// captured now, and another thread's hipStreamPerThread.  A thread may ask while
// others capture in global mode only in relaxed mode.
hipError_t query_slot(const Slot& s) {
  if (s.stream == hipStreamPerThread) return hipErrorNotReady;
  int current = 0;
  hipError_t e = hipGetDevice(&current);
  if (e != hipSuccess) return e;
  if (current != s.device && (e = hipSetDevice(s.device)) != hipSuccess) return e;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  e = hipThreadExchangeStreamCaptureMode(&mode);
  if (e == hipSuccess) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    e = hipStreamIsCapturing(s.stream, &status);
    if (e == hipErrorStreamCaptureImplicit || (e == hipSuccess && status != hipStreamCaptureStatusNone))
      e = hipErrorNotReady;
    else
      e = hipStreamQuery(s.stream);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
  (void)hipGetLastError();  // "not ready" is no error of a later call's
  if (current != s.device) (void)hipSetDevice(current);
  return e;
}

// Waits until the slot's pending upload has read it.  The stream may have any
// amount of work before the upload, but one that has failed or is gone never
// gets there: a wait of seconds asks the runtime.
int wait_slot(Slot& s) {
  const uint32_t* done = reinterpret_cast<const uint32_t*>(s.host + s.words_at);
  size_t n_read = 0;
  auto read = [&] {
    while (n_read < s.n_words && __atomic_load_n(done + n_read, __ATOMIC_ACQUIRE) != 0) ++n_read;
    return n_read == s.n_words;
  };
  constexpr std::chrono::seconds kAskEvery(2);
  std::chrono::steady_clock::time_point ask = std::chrono::steady_clock::time_point::max();
  for (int spins = 0; !read(); spins += spins < 1000) {
    if (spins < 1000) continue;
    const std::chrono::steady_clock::time_point now = std::chrono::steady_clock::now();
    if (ask == std::chrono::steady_clock::time_point::max()) ask = now + kAskEvery;
    if (now >= ask) {
      const hipError_t e = query_slot(s);
      if (e != hipErrorNotReady && !read()) {
        // Whether anything still reads the memory is unknown: it is left.
        s.host = nullptr;
        s.mapped = nullptr;
        s.cap = s.n_words = 0;
        return fail(CP_ERR_HIP, std::string("cp_attn_partial: an earlier table upload did not run: ") + hipGetErrorString(e));
      }
      ask = now + kAskEvery;
    }
    std::this_thread::sleep_for(std::chrono::microseconds(10));
  }
  s.n_words = 0;
  return CP_OK;
}

int stage_and_copy(const Plan& plan, const Layout& lay, void* dst, hipStream_t stream) {
  const size_t bytes = lay.pieces;  // the tables; a multiple of 256
  if (capturing(stream)) {
    std::vector<unsigned char> host(bytes);
    pack_tables(plan, lay, host.data());
    return cpattn::launch_upload(dst, host.data(), bytes, stream);
  }
  const size_t n_words = upload_blocks(bytes);
  Slot& s = g_slots[g_next_slot.fetch_add(1) % kSlots];
  std::lock_guard<std::mutex> lock(s.mu);
  int st = wait_slot(s);
  if (st != CP_OK) return st;
  hipError_t e = hipGetDevice(&s.device);
  if (e != hipSuccess) return fail(CP_ERR_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
  s.stream = stream;
  if (s.cap < bytes + 4 * n_words) {
    if (s.host) (void)hipHostFree(s.host);
    s.host = nullptr;
    s.mapped = nullptr;
    s.cap = 0;
    const size_t cap = std::max<size_t>(bytes + 4 * n_words, 64 * 1024);
    void* host = nullptr;
    e = hipHostMalloc(&host, cap, hipHostMallocMapped | hipHostMallocPortable | hipHostMallocCoherent);
    if (e != hipSuccess) return fail(CP_ERR_HIP, std::string("hipHostMalloc (staging): ") + hipGetErrorString(e));
    s.host = static_cast<unsigned char*>(host);
    e = hipHostGetDevicePointer(&s.mapped, s.host, 0);
    if (e != hipSuccess) return fail(CP_ERR_HIP, std::string("hipHostGetDevicePointer (staging): ") + hipGetErrorString(e));
    s.cap = cap;
  }
  pack_tables(plan, lay, s.host);
  std::memset(s.host + bytes, 0, 4 * n_words);
  st = cpattn::launch_upload(dst, s.mapped, bytes, stream);
  if (st != CP_OK) return st;
  s.words_at = bytes;
  s.n_words = n_words;
  return CP_OK;
}

}  // namespace

extern "C" size_t cp_attn_partial_workspace_size(const cp_partial_desc* descs, int32_t n_descs,
                                                 int32_t n_heads_q, int32_t n_heads_kv) {
  size_t total = 0;
  const int st = guarded([&]() -> int {
    Plan plan;
    const int s = build_plan(descs, n_descs, n_heads_q, n_heads_kv, kTargetPieces, &plan);
    if (s == CP_OK) total = layout_of(plan).total;
    return s;
  });
  if (st != CP_OK) return 0;
  clear_error();
  return total;
}

extern "C" int cp_attn_partial(const cp_partial_desc* descs, int32_t n_descs, int32_t n_heads_q,
                               int32_t n_heads_kv, int32_t head_dim, float softmax_scale, void* workspace,
                               size_t workspace_bytes, void* stream) {
  return guarded([&]() -> int {
    if (head_dim != CP_HEAD_DIM) return fail(CP_ERR_UNSUPPORTED, "cp_attn_partial: head_dim must be 128");
    if (!(softmax_scale == softmax_scale)) return fail(CP_ERR_INVALID, "cp_attn_partial: softmax_scale is NaN");
    Plan plan;
    Layout lay;
    size_t wanted = 0;
    int st = build_plan_within(descs, n_descs, n_heads_q, n_heads_kv, workspace ? workspace_bytes : SIZE_MAX, &plan,
                               &lay, &wanted);
    if (st != CP_OK) return st;
    if (plan.items.empty()) {
      clear_error();
      return CP_OK;
    }
    if (!workspace) return fail(CP_ERR_INVALID, "cp_attn_partial: workspace is NULL");
    if (!aligned(workspace, 256)) return fail(CP_ERR_INVALID, "cp_attn_partial: workspace must be 256-byte aligned");
    if (workspace_bytes < lay.total)
      return fail(CP_ERR_CAPACITY, "cp_attn_partial: workspace needs " + std::to_string(wanted) + " bytes");
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.f / std::sqrt((float)head_dim);
    PartialParams p =
        partial_params(plan, lay, static_cast<unsigned char*>(workspace), n_heads_q, n_heads_kv, scale);
    InlineTables inl;
    if (pack_inline(plan, &inl)) {
      p.inl = &inl;
    } else {
      // Only the tables are uploaded; the piece slots are written by the kernel.
      st = stage_and_copy(plan, lay, workspace, (hipStream_t)stream);
      if (st != CP_OK) return st;
    }
    st = launch_partial(p, stream);
    if (st == CP_OK) clear_error();
    return st;
  });
}

extern "C" int cp_attn_merge(int32_t n_parts, const float* const* o_parts, const float* const* lse_parts,
                             int64_t n_tokens, int32_t n_heads, int32_t head_dim, void* o_out, int32_t out_bf16,
                             float* lse_out, const cp_rank_plan* restore, void* stream) {
  return guarded([&]() -> int {
    if (head_dim != CP_HEAD_DIM) return fail(CP_ERR_UNSUPPORTED, "cp_attn_merge: head_dim must be 128");
    if (n_parts < 1 || n_parts > CP_MAX_MERGE_PARTS) return fail(CP_ERR_INVALID, "cp_attn_merge: n_parts must be 1..16");
    if (!o_parts || !lse_parts) return fail(CP_ERR_INVALID, "cp_attn_merge: o_parts/lse_parts is NULL");
    if (n_tokens < 0 || n_heads < 1) return fail(CP_ERR_INVALID, "cp_attn_merge: n_tokens < 0 or n_heads < 1");
    if (out_bf16 != 0 && out_bf16 != 1) return fail(CP_ERR_INVALID, "cp_attn_merge: out_bf16 must be 0 or 1");
    MergeParams p;
    std::memset(&p, 0, sizeof(p));
    if (n_tokens > 0) {
      for (int i = 0; i < n_parts; ++i) {
        if (!o_parts[i] || !lse_parts[i]) return fail(CP_ERR_INVALID, "cp_attn_merge: NULL partial pointer");
        if (!aligned(o_parts[i], 16) || !aligned(lse_parts[i], 4))
          return fail(CP_ERR_INVALID, "cp_attn_merge: partial O must be 16-byte, LSE 4-byte aligned");
        p.o[i] = o_parts[i];
        p.lse[i] = lse_parts[i];
      }
      if (!o_out) return fail(CP_ERR_INVALID, "cp_attn_merge: o_out is NULL");
      if (!aligned(o_out, 16)) return fail(CP_ERR_INVALID, "cp_attn_merge: o_out must be 16-byte aligned");
      if (lse_out && !aligned(lse_out, 4)) return fail(CP_ERR_INVALID, "cp_attn_merge: lse_out must be 4-byte aligned");
    }
    if (restore) {
      cp_rank_plan ref;
      if (make_plan(restore->prefix_len, restore->new_len, restore->C, restore->rank, &ref) != CP_OK ||
          !plan_equal(ref, *restore))
        return fail(CP_ERR_INVALID, "cp_attn_merge: restore plan does not match cp_shard_plan");
      if (restore->n_rows != n_tokens) return fail(CP_ERR_INVALID, "cp_attn_merge: n_tokens != restore->n_rows");
      p.restore = 1;
      p.first_len = restore->chunk[0].q_len;
      p.first_dst = restore->chunk[0].q_begin - restore->prefix_len;
      p.second_dst = restore->chunk[1].q_begin - restore->prefix_len;
    }
    p.n_parts = n_parts;
    p.n_heads = n_heads;
    p.n_tokens = n_tokens;
    p.o_out = o_out;
    p.lse_out = lse_out;
    p.out_bf16 = out_bf16;
    int st = launch_merge(p, stream);
    if (st == CP_OK) clear_error();
    return st;
  });
}
