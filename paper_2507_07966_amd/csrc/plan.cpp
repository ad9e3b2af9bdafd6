// Host side of the library: descriptor validation, the work lists of the two attention
// passes, workspace layout, plan lifetime and schedule introspection.
//
// Shapes follow the paper's rollout-and-prefill description (Sec. 4.2: G responses per
// question; Sec. 5.1: one cached video embedding shared by all rollouts; Sec. 5.2: prefill
// of every rollout): a shared prefix of P tokens and G ragged suffixes packed back to back.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <initializer_list>
#include <new>
#include <utility>

#include "common.h"

using pa::WorkItem;

namespace {

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int validate(const prefix_attn_desc_t* d) {
  if (d->num_q_heads < 1 || d->num_kv_heads < 1 || d->num_q_heads % d->num_kv_heads != 0) return PA_ERR_SHAPE;
  if (d->head_dim < 1 || d->prefix_len < 0 || d->num_rollouts < 1) return PA_ERR_SHAPE;
  if (!(d->softmax_scale > 0.0f) || !std::isfinite(d->softmax_scale)) return PA_ERR_SHAPE;
  if (d->device < -1) return PA_ERR_SHAPE;
  if (d->prefix_len > (int64_t)1 << 30) return PA_ERR_SHAPE;  // key indices are 32-bit in the kernels
  if (!d->suffix_lens) return PA_ERR_NULL;
  int64_t T = 0;
  for (int g = 0; g < d->num_rollouts; ++g) {
    if (d->suffix_lens[g] < 1) return PA_ERR_SHAPE;
    T += d->suffix_lens[g];
  }
  const int64_t group = d->num_q_heads / d->num_kv_heads;
  // stacked row indices (S_g * group) and packed rows times heads must fit 32-bit arithmetic
  for (int g = 0; g < d->num_rollouts; ++g)
    if ((int64_t)d->suffix_lens[g] * group > (int64_t)1 << 30) return PA_ERR_SHAPE;
  if (T * d->num_q_heads > (int64_t)1 << 31) return PA_ERR_SHAPE;
  if (d->dtype != PA_F32 && d->dtype != PA_BF16) return PA_ERR_UNSUPPORTED;
  if (d->head_dim != 64 && d->head_dim != 128) return PA_ERR_UNSUPPORTED;
  if (d->dtype == PA_BF16) {  // the bf16 kernels address a key set (the prefix, one rollout) with 32-bit byte offsets
    const int64_t row_bytes = (int64_t)d->num_kv_heads * d->head_dim * 2, limit = (int64_t)1 << 31;
    if (d->prefix_len * row_bytes >= limit) return PA_ERR_UNSUPPORTED;
    for (int g = 0; g < d->num_rollouts; ++g)
      if (d->suffix_lens[g] * row_bytes >= limit) return PA_ERR_UNSUPPORTED;
  }
  return PA_OK;
}

// Lays per-kv-head lists out so that workgroup n (dispatched to XCD n % num_xcd) always belongs to the same
// kv head: each head owns num_xcd / Hkv XCDs, whose L2 then serves that head's tiles to all the workgroups
// walking them together.  Slots without an item hold `pad` (the workgroup exits).  When the XCD count is not
// a multiple of the head count the lists are simply concatenated.
template <class Item>
void interleave_over_xcds(const std::vector<std::vector<Item>>& per_head, int num_xcd, const Item& pad,
                          std::vector<Item>& out) {
  const int Hkv = (int)per_head.size();
  out.clear();
  if (Hkv <= num_xcd && num_xcd % Hkv == 0) {
    size_t per = 0;
    for (const auto& v : per_head) per = std::max(per, v.size());
    const int xper = num_xcd / Hkv;  // XCDs per kv head
    const size_t qlen = (per + xper - 1) / xper;
    out.assign(qlen * num_xcd, pad);
    for (int x = 0; x < num_xcd; ++x) {
      const int c = x / xper, sub = x % xper;
      for (size_t k = 0; k * xper + sub < per_head[c].size(); ++k) out[k * num_xcd + x] = per_head[c][k * xper + sub];
    }
  } else {
    for (const auto& v : per_head) out.insert(out.end(), v.begin(), v.end());
  }
}

const WorkItem PAD_ITEM{-1, 0, 0, 0, 0, 0, 0, 0};

// Prefix pass: every (kv head, rollout, block of stacked rows) sweeps all P keys.  Workgroup n
// runs on XCD n % 8 and each XCD has a private L2, so the list is interleaved such that one kv
// head's items land on a fixed subset of XCDs and walk the prefix K/V tiles together: the
// tiles are then fetched from HBM about once per XCD subset instead of once per workgroup.
//
// A call with few rows (a short prompt over a long video, say) has fewer row blocks than the
// chip has CUs.  The prefix keys are then cut into `key_splits` contiguous ranges of whole
// tiles, one item per (row block, range), each leaving its own fp32 partial; the merge combines
// them with the suffix partial.  Items of one range are adjacent so they share its tiles in L2.
void build_prefix_items(prefix_attn_plan_t& p) {
  std::vector<WorkItem>& out = p.items[0];
  out.clear();
  p.key_splits = 1;
  const int Hkv = p.desc.num_kv_heads;
  const int P = (int)p.desc.prefix_len;
  if (P == 0) return;
  int64_t blocks = 0;
  for (int g = 0; g < p.desc.num_rollouts; ++g)
    blocks += ((int64_t)p.lens[g] * p.group + pa::ROWS_PER_ITEM - 1) / pa::ROWS_PER_ITEM;
  blocks *= Hkv;
  if (p.desc.dtype == PA_BF16) {  // one round of workgroups, at least 8 tiles per range
    const int64_t fit = p.num_cu / blocks, by_len = p.tiles_prefix / 8;
    p.key_splits = (int32_t)std::max<int64_t>(1, std::min<int64_t>({fit, by_len, PA_MAX_PARTIALS - 1}));
  }
  const int tiles_per_split = (p.tiles_prefix + p.key_splits - 1) / p.key_splits;
  p.key_splits = (p.tiles_prefix + tiles_per_split - 1) / tiles_per_split;  // no empty range
  const int KS = p.key_splits;
  std::vector<std::vector<WorkItem>> per_head(Hkv);
  for (int c = 0; c < Hkv; ++c)
    for (int s = 0; s < KS; ++s) {
      const int key0 = std::min(s * tiles_per_split * pa::KEYS_PER_TILE, P);
      const int key1 = std::min((s + 1) * tiles_per_split * pa::KEYS_PER_TILE, P);
      for (int g = 0; g < p.desc.num_rollouts; ++g) {
        const int nrows = p.lens[g] * p.group;
        for (int row0 = 0; row0 < nrows; row0 += pa::ROWS_PER_ITEM)
          per_head[c].push_back({g, row0, c, key1 - key0, key0, s, 0, 0});
      }
    }
  interleave_over_xcds(per_head, p.num_xcd, PAD_ITEM, out);
}

// Suffix pass: a block of stacked rows needs the rollout's keys 0..(position of its last row).
// Items are issued longest first so the ragged, triangular work packs well.
void build_suffix_items(prefix_attn_plan_t& p) {
  std::vector<WorkItem>& out = p.items[1];
  out.clear();
  for (int c = 0; c < p.desc.num_kv_heads; ++c)
    for (int g = 0; g < p.desc.num_rollouts; ++g) {
      const int nrows = p.lens[g] * p.group;
      for (int row0 = 0; row0 < nrows; row0 += pa::ROWS_PER_ITEM) {
        const int last_row = std::min(row0 + pa::ROWS_PER_ITEM, nrows) - 1;
        out.push_back({g, row0, c, last_row / p.group + 1, 0, 0, 0, 0});
      }
    }
  std::stable_sort(out.begin(), out.end(), [](const WorkItem& a, const WorkItem& b) { return a.nkeys > b.nkeys; });
}

// fp32: the suffix list's blocks in pieces of 16 or 32 rows, one workgroup each.  One workgroup of 8 wavefronts runs per CU
// at a time, so a launch takes ceil(workgroups / CUs) rounds, and a round of 32-row workgroups takes 1.5 to 1.65 times one
// of 16-row workgroups (measured, 8 / 2 heads of 128 channels, 1,000 prefix keys, us with 16 / 32 rows: 370 blocks of 16
// rows 72 / 62, 600 blocks 106 / 104, 1,024 blocks 152 / 121, 2,400 blocks 352 / 273; up to 256 blocks 16 rows take one
// round and 32 rows leave half the CUs idle).
// Only pieces that hold rows are listed.  (A workgroup for each of the 16 pieces of a 256-row item ran empty ones where
// rollouts are short, and left the work to one XCD, as workgroup n runs on XCD n % 8: 1,000 one-token rollouts, 1,000 prefix
// keys, 8 / 2 heads of 128: forward 2,770 -> 240 us, backward 5,210 -> 560.)
// With at most 128 keys a block on average, sharing them between 8 wavefronts leaves most of those without work; where that
// ends earlier (us per round of 8 / of 1 wavefront a block, from calls of one kind of block) a block then gets one
// wavefront, 8 blocks run per CU: 20,000 one-token rollouts, 4 heads of 64, no prefix 888 -> 93 us; 10,000 of 8 tokens,
// 8 / 2 heads of 128 671 -> 197 us.
void build_f32_blocks(prefix_attn_plan_t& p) {
  for (auto& v : p.f32_blocks) v.clear();
  p.f32_rows = 16;
  p.f32_waves = 8;
  if (p.desc.dtype != PA_F32) return;
  auto pieces = [&](int rows, std::vector<WorkItem>& out) {
    for (const WorkItem& it : p.items[1]) {
      const int end = std::min(it.row0 + pa::ROWS_PER_ITEM, p.lens[it.g] * p.group);
      for (int row0 = it.row0; row0 < end; row0 += rows) out.push_back({it.g, row0, it.c, 0, 0, 0, 0, 0});
    }
  };
  pieces(16, p.f32_blocks[1]);
  pieces(32, p.f32_blocks[0]);
  auto rounds = [&](size_t blocks, int at_once) { return (double)((blocks + at_once - 1) / at_once); };
  const double rounds16 = rounds(p.f32_blocks[1].size(), p.num_cu), rounds32 = rounds(p.f32_blocks[0].size(), p.num_cu);
  if (3 * rounds32 <= 2 * rounds16) p.f32_rows = 32;
  const double prefix_blocks = (double)((p.desc.prefix_len + 15) / 16);  // of 16 keys
  double sum = 0.0, longest = 0.0;
  for (const WorkItem& it : p.f32_blocks[1]) {
    const double n = prefix_blocks + it.row0 / p.group / 16 + 1;
    sum += n;
    longest = std::max(longest, n);
  }
  const double mean = sum / (double)p.f32_blocks[1].size();
  const double shared = std::min(rounds16, 1.55 * rounds32) * (5.0 + 0.45 * mean);
  const double alone = std::max(rounds(p.f32_blocks[1].size(), 8 * p.num_cu) * (2.0 + 2.6 * mean), 2.0 + 2.6 * longest);
  if (mean <= 8.0 && alone < shared) {
    p.f32_rows = 16;
    p.f32_waves = 1;
  }
  if (p.f32_rows == 16) p.f32_blocks[0] = p.f32_blocks[1];
}

// Backward, dQ pass: the suffix pass's blocks of rows (longest first); each sweeps the prefix and
// then its own keys.  With key splits (few rows, see build_prefix_items) a block appears once per
// prefix key range; split 0 also sweeps the own keys, and the fp32 partial dQ are added afterwards.
void build_dq_items(prefix_attn_plan_t& p) {
  p.dq_items.clear();
  const int P = (int)p.desc.prefix_len;
  const int KS = p.key_splits;
  const int tiles_per_split = (p.tiles_prefix + KS - 1) / KS;  // the ranges of build_prefix_items
  for (int s = 0; s < KS; ++s) {
    const int key0 = std::min(s * tiles_per_split * pa::KEYS_PER_TILE, P);
    const int key1 = std::min((s + 1) * tiles_per_split * pa::KEYS_PER_TILE, P);
    for (const WorkItem& it : p.items[1])
      p.dq_items.push_back({it.g, it.row0, it.c, s == 0 ? it.nkeys : 0, key0, s, key1 - key0, 0});
  }
  // An unsplit prefix: lay the blocks out over the XCDs by kv head like the prefix pass, so that the
  // workgroups of an XCD walk the same K, V and K^T tiles together (-0.4 % at a 32K prefix, -1.5 % at 230K).
  const int Hkv = p.desc.num_kv_heads;
  if (KS == 1 && P > 0 && Hkv <= p.num_xcd && p.num_xcd % Hkv == 0) {
    std::vector<std::vector<WorkItem>> per_head(Hkv);
    for (const WorkItem& it : p.dq_items) per_head[it.c].push_back(it);  // longest first inside a kv head
    interleave_over_xcds(per_head, p.num_xcd, PAD_ITEM, p.dq_items);
  }
}

// Forward sweep (one pass over [prefix | own keys] per block of rows): the prefix dominates, so the blocks are
// laid out like the prefix pass's (one kv head per subset of XCDs, sharing its K/V tiles in that L2), and
// inside a kv head longest first.
void build_sweep_items(prefix_attn_plan_t& p) {
  p.sweep_items.clear();
  const int Hkv = p.desc.num_kv_heads;
  const int P = (int)p.desc.prefix_len;
  if (P == 0 || p.key_splits != 1 || p.desc.dtype != PA_BF16 || p.tiles_prefix > pa::SWEEP_MAX_PREFIX_TILES) return;
  std::vector<std::vector<WorkItem>> per_head(Hkv);
  for (const WorkItem& it : p.items[1]) per_head[it.c].push_back({it.g, it.row0, it.c, it.nkeys, 0, 0, P, 0});  // sorted already
  interleave_over_xcds(per_head, p.num_xcd, PAD_ITEM, p.sweep_items);
}

// When the last of `cost` (whole units) ends, the longest first on whichever of `at_once` workers is free; a value of at least
// `enough` if that is certain beforehand or on the way.  Sorts `cost`.
int list_schedule(std::vector<int>& cost, int at_once, double enough) {
  int64_t sum = 0;
  int longest = 0;
  for (int t : cost) {
    sum += t;
    longest = std::max(longest, t);
  }
  if ((int)cost.size() <= at_once) return longest;
  const int least = std::max(longest, (int)std::min<int64_t>((sum + at_once - 1) / at_once, INT32_MAX));
  if (least >= enough) return least;
  if (!std::is_sorted(cost.begin(), cost.end(), std::greater<int>())) std::sort(cost.begin(), cost.end(), std::greater<int>());
  // a heap of the times at which the workers are free, the earliest at the top
  std::vector<int> free(cost.begin(), cost.begin() + at_once);
  std::reverse(free.begin(), free.end());  // ascending: a heap already
  int end = longest;
  for (size_t n = at_once; n < cost.size(); ++n) {
    const int t = free[0] + cost[n];
    end = std::max(end, t);
    if (end >= enough) return end;
    size_t at = 0;
    for (size_t child; (child = 2 * at + 1) < free.size(); at = child) {
      if (child + 1 < free.size() && free[child + 1] < free[child]) ++child;
      if (free[child] >= t) break;
      free[at] = free[child];
    }
    free[at] = t;
  }
  return end;
}

// Into how many ranges of key tiles to cut each block of rows so that one workgroup per CU ends early.  Whole blocks take
// ceil(blocks / CUs) rounds, and the last one may hold a single block; a call of few rows has fewer blocks than CUs.
struct CutCosts {
  double tile_us;    // one key tile of a block
  double item_tiles; // an item's start and end, in tiles
  double slot_us;    // a fp32 partial result written and read
  double launch_us;  // the launch that adds them
};
// `tiles`: key tiles of the blocks of one kv head, longest first; `most`: ranges they can be cut into; `cus`: CUs that run
// them; `whole_us`: what the uncut blocks cost (< 0: as estimated here).  Candidates are compared by list scheduling: up to
// one block per CU, no range longer than 1 / n of the longest block; more blocks, those beyond full rounds cut into n ranges
// each, so that they are spread over all CUs.  Empty: leave the blocks whole.
std::vector<int> cut_blocks(const std::vector<int>& tiles, const std::vector<int>& most, int cus, const CutCosts& c,
                            double whole_us, size_t max_slots) {
  const int N = (int)tiles.size(), rest = N % cus;
  std::vector<int> cost;  // tiles
  std::vector<int> pieces(N, 1), chosen;
  const int item_tiles = (int)c.item_tiles;
  auto estimate = [&](double enough_us) {
    size_t slots = 0, items = 0;
    for (int b = 0; b < N; ++b) {
      if (pieces[b] > 1) slots += pieces[b];
      items += pieces[b];
    }
    if (slots > 0 && items > (size_t)N + 2 * cus) return 1e30;  // two ranges a CU even out what there is to even out
    if (slots > max_slots) return 1e30;
    cost.clear();
    for (int b = 0; b < N; ++b) cost.insert(cost.end(), pieces[b], (tiles[b] + pieces[b] - 1) / pieces[b] + item_tiles);
    const double extra = slots ? (double)slots * c.slot_us + c.launch_us : 0.0;
    return c.tile_us * list_schedule(cost, cus, (enough_us - extra) / c.tile_us) + extra;
  };
  double sum = 0.0;
  for (int t : tiles) sum += t + c.item_tiles;
  double best_us = whole_us >= 0.0 ? whole_us : 0.95 * estimate(1e30);
  if (c.tile_us * sum / cus + c.launch_us >= best_us) return chosen;  // nothing to gain
  auto consider = [&]() {
    const double us = estimate(best_us);
    if (us < best_us) {
      best_us = us;
      chosen = pieces;
    }
  };
  for (int n = 2; n <= PA_MAX_PARTIALS; n += N <= cus ? 1 : n) {
    const int limit = (tiles.front() + n - 1) / n;
    for (int b = 0; b < N; ++b)
      pieces[b] = std::min(most[b], N <= cus ? (tiles[b] + limit - 1) / limit : b < rest ? n : 1);
    consider();
  }
  return chosen;
}

// CUs that run the blocks of one kv head when the lists are laid out by interleave_over_xcds, and whether they are.
bool heads_apart(const prefix_attn_plan_t& p) { return p.desc.num_kv_heads <= p.num_xcd && p.num_xcd % p.desc.num_kv_heads == 0; }

pa::RangeSum range_sum(const prefix_attn_plan_t& p, const WorkItem& it, int slot0, int n) {
  return {p.cu[it.g], it.row0, it.c, std::min(pa::ROWS_PER_ITEM, p.lens[it.g] * p.group - it.row0), slot0, n};
}

// Cuts the blocks of items[1] into `pieces` ranges of their tile sequence [prefix | own keys] (of the first kv head's
// blocks, or of all: see heads_apart), numbers the slots of the cut ones and lays the items out: longest first, ranges of
// equal length in the order of their keys, so that neighbours share tiles in L2.  With `diagonal` no range starts inside
// the own keys after the position of the block's first row.
void lay_out_ranges(const prefix_attn_plan_t& p, const std::vector<int>& pieces, bool diagonal, std::vector<WorkItem>& out,
                    std::vector<pa::RangeSum>& sums, int32_t& slots) {
  const int P = (int)p.desc.prefix_len, tp = p.tiles_prefix, BN = pa::KEYS_PER_TILE, Hkv = p.desc.num_kv_heads;
  const bool apart = heads_apart(p);
  struct Range { int tiles; WorkItem it; };
  std::vector<std::vector<Range>> per_head(apart ? Hkv : 1);
  std::vector<size_t> next(Hkv, 0);  // the blocks of every kv head stand in the same order
  for (const WorkItem& it : p.items[1]) {
    const int n = pieces[next[apart ? it.c : 0]++];
    const int total = tp + (it.nkeys + BN - 1) / BN, legal = diagonal ? tp + it.row0 / p.group / BN : total;
    auto cut = [&](int i) {  // first tile of range i
      return i == n ? total : std::max(i, std::min((int)((int64_t)total * i / n), legal - (n - 1 - i)));
    };
    if (n > 1)
      sums.push_back(range_sum(p, it, slots, n));
    for (int i = 0; i < n; ++i) {
      const int t0 = cut(i), t1 = cut(i + 1);
      const int p0 = std::min(std::min(t0, tp) * BN, P), p1 = std::min(std::min(t1, tp) * BN, P);
      const int o0 = std::max(t0 - tp, 0) * BN, o1 = std::min(std::max(t1 - tp, 0) * BN, it.nkeys);
      const int slot = n > 1 ? slots++ : -1;
      per_head[apart ? it.c : 0].push_back(
          {t1 - t0, {it.g, it.row0, it.c, std::max(o1 - o0, 0), p1 > p0 ? p0 : 0, slot, p1 - p0, o0}});
    }
  }
  std::vector<std::vector<WorkItem>> lists(per_head.size());
  for (size_t c = 0; c < per_head.size(); ++c) {
    std::stable_sort(per_head[c].begin(), per_head[c].end(), [](const Range& a, const Range& b) {
      return a.tiles != b.tiles ? a.tiles > b.tiles : a.it.key0 < b.it.key0;
    });
    for (const Range& r : per_head[c]) lists[c].push_back(r.it);
  }
  interleave_over_xcds(lists, p.num_xcd, PAD_ITEM, out);
}

// The launch list of the bf16 dQ pass.  With key splits (few rows) the dQ list's items, their partials numbered block by
// block; otherwise blocks that would leave CUs idle are cut as in the forward's sweep (costs at D = 128 (64): 2.7 (1.2) us
// per key tile, 4 tiles for an item's start and end).  The fp32 partials of a cut block are added afterwards.  5,377
// prefix keys, 5 rollouts of 37 ... 1,901 tokens, 14 / 2 heads of 64: 158 -> 117 us plus 8 us for the sums.
void build_dq_launch(prefix_attn_plan_t& p) {
  p.dq_launch.clear();
  p.dq_sums.clear();
  p.dq_slots = 0;
  if (p.desc.dtype != PA_BF16) return;
  const int BN = pa::KEYS_PER_TILE, KS = p.key_splits;
  if (KS > 1) {
    const size_t blocks = p.items[1].size();  // the dQ list holds them once per split, in this order
    for (const WorkItem& it : p.items[1]) {
      p.dq_sums.push_back(range_sum(p, it, p.dq_slots, KS));
      p.dq_slots += KS;
    }
    p.dq_launch = p.dq_items;
    for (size_t n = 0; n < p.dq_launch.size(); ++n) p.dq_launch[n].split += p.dq_sums[n % blocks].slot0;
    return;
  }
  const bool apart = heads_apart(p);
  const int heads = apart ? p.desc.num_kv_heads : 1;
  if (2 * p.items[1].size() > (size_t)p.num_cu && p.items[1].size() <= 2 * (size_t)p.num_cu) {  // fewer: key splits
    std::vector<int> tiles, most;
    for (const WorkItem& it : p.items[1])
      if (!apart || it.c == 0) {
        tiles.push_back(p.tiles_prefix + (it.nkeys + BN - 1) / BN);
        most.push_back(std::min(PA_MAX_PARTIALS, tiles.back()));
      }
    const CutCosts costs{p.desc.head_dim == 128 ? 2.7 : 1.2, 4.0,
                         heads * (double)pa::ROWS_PER_ITEM * p.desc.head_dim * 4 * 2 / 4e6, 5.0};
    const std::vector<int> pieces = cut_blocks(tiles, most, p.num_cu / heads, costs, -1.0, ~(size_t)0);
    if (!pieces.empty()) return lay_out_ranges(p, pieces, false, p.dq_launch, p.dq_sums, p.dq_slots);
  }
  p.dq_launch = p.dq_items;
  for (WorkItem& it : p.dq_launch) it.split = -1;
}

// Forward, the sweep over [prefix | own keys] with some blocks of rows cut into ranges (cut_blocks), one launch and one
// merge of the cut blocks.  Costs measured at D = 128 (64): 1.56 (0.9) us per key tile, 5 tiles' time for an item's start
// and end, partials written and read at 4 TB/s, 8 us for the merge launch (4 us of its own; a small call was bound
// by the rate of launches while it also had an image pre-pass and a careful launch: with 5 here calls of 5 to 12 prefix tiles were
// cut, 20.5 -> 22.5 us).  For short calls (mark_short_calls), which have neither, 8 us is too much: 128 tokens, 28 / 4 heads of 128
// (14 / 2 of 64), whole, as this rule has them, and cut as 4 us would: 6 prefix tiles 21.0 and 19.2 us, 8 tiles 23.8 and 20.4 (16.1 and
// 12.6), 10 tiles of 64 channels 18.0 and 12.7; up to 4 tiles whole is as fast or faster, from 12 tiles on both cut alike
// (12 tiles 29.2 whole, 22.2 cut).  Up to two rounds of whole blocks: beyond that the last round is at most a third of the call, its CUs run at a higher clock and the others' spread fills it.
// 128 tokens, 28 / 4 heads of 128, 1,024 prefix keys (16 blocks, 6 ranges each): passes 37 -> 18 us, the whole call
// with its LSE 45.3 -> 27.5 us.  88 blocks of a kv head for its 128 CUs (5,377
// prefix keys, 5 rollouts of 37 ... 1,901 tokens, 14 / 2 heads of 64), two ranges each: pass 114 -> 84 us, merge 8 us.
// With few rows the alternative is the prefix pass over key ranges (one partial of every row a range), a suffix pass and the
// n-way merge.  Cuts win (7,922 keys, 4 rollouts of up to 9 tokens, 4 heads of 128: 32 us, else 44) unless the 64 MiB
// workspace has too little room for the 256-row slots of short blocks; then the two are compared as they fit: 54,411 keys, 6
// rollouts of up to 19 tokens, 4 heads of 128: 392 us in the cuts that fit, 166 with 10 key ranges of the prefix.
// Cuts inside the own keys stay at or before the position of the block's first row: every row then sees the first key
// of every range, so no partial is empty.
void build_range_items(prefix_attn_plan_t& p, size_t fixed_bytes, size_t slot_bytes) {
  p.range_items.clear();
  p.range_sums.clear();
  p.range_slots = 0;
  const int tp = p.tiles_prefix, BN = pa::KEYS_PER_TILE, Hkv = p.desc.num_kv_heads;
  if (p.desc.dtype != PA_BF16 || p.items[1].size() > 2 * (size_t)p.num_cu) return;
  const bool apart = heads_apart(p);
  std::vector<WorkItem> blocks;  // of the first kv head, or of all
  for (const WorkItem& it : p.items[1])
    if (!apart || it.c == 0) blocks.push_back(it);
  const int heads = apart ? Hkv : 1;
  std::vector<int> tiles, most;
  for (const WorkItem& it : blocks) {
    tiles.push_back(tp + (it.nkeys + BN - 1) / BN);
    most.push_back(std::min(PA_MAX_PARTIALS, std::min(tiles.back(), tp + it.row0 / p.group / BN + 1)));
  }
  const size_t bytes_per_slot = (size_t)pa::ROWS_PER_ITEM * (p.desc.head_dim + 1) * sizeof(float);
  const CutCosts costs{p.desc.head_dim == 128 ? 1.56 : 0.9, 5.0, heads * (double)bytes_per_slot * 2 / 4e6, 8.0};
  // what fitted the library's own workspace keeps fitting
  const size_t had = (size_t)(p.key_splits + 1) * slot_bytes;
  const size_t room = fixed_bytes + had <= PA_STATIC_SCRATCH_BYTES ? PA_STATIC_SCRATCH_BYTES - fixed_bytes : ~(size_t)0;
  // flags of at most two ranges a CU beside the blocks, and the pads of the layout over the XCDs
  const size_t flags = (blocks.size() * heads + 2 * (size_t)p.num_cu + p.num_xcd) * pa::WAVES_PER_ITEM * sizeof(int32_t) + 4 * 256;
  size_t max_slots = room == ~(size_t)0 ? room : room <= flags ? 0 : (room - flags) / (bytes_per_slot + 256) / heads;
  const int KS = p.key_splits;
  const double whole_us = KS > 1 ? 1e30 : -1.0;
  std::vector<int> pieces = cut_blocks(tiles, most, p.num_cu / heads, costs, whole_us, KS > 1 ? ~(size_t)0 : max_slots);
  size_t slots = 0;
  for (int n : pieces) slots += n > 1 ? n : 0;
  if (KS > 1 && slots > max_slots) {
    const double rows = (double)p.T * p.desc.num_q_heads;
    const double partials_us = (KS + 1) * rows * (p.desc.head_dim + 1) * 4 * 2 / 4e6;
    CutCosts short_blocks = costs;  // of a slot only the block's rows are written and read
    short_blocks.slot_us *= rows / ((double)p.items[1].size() * pa::ROWS_PER_ITEM);
    const double other_us = costs.tile_us * ((tp + KS - 1) / KS + tiles.front() - tp + 2 * costs.item_tiles) + partials_us +
                            2 * costs.launch_us;
    pieces = cut_blocks(tiles, most, p.num_cu / heads, short_blocks, other_us, max_slots);
  }
  if (pieces.empty()) return;

  lay_out_ranges(p, pieces, true, p.range_items, p.range_sums, p.range_slots);
}

// Whole bf16 calls of few key tiles (those of the longest item, times the rounds of items) run as one launch (and the merge of cut
// blocks): V is read as it is instead of from images, and the workgroup itself redoes an item whose scores leave the common
// kernel's range, so neither the image pre-pass nor the launch of the careful kernel is needed.  What these cost, 4 to 8 us, against
// transposed reads of V (two for one, and 3 to 4 % of the pass): forward and LSE export, 28 / 4 heads of 128, 12 blocks of 6 tiles
// 29.6 -> 22.2 us, 18 tiles 53.0 -> 49.5, 72 tiles 121.7 -> 118.0, 126 tiles 114.4 -> 112.1, 136 tiles 204.7 -> 202.8, 264 tiles
// 378.5 -> 381.2, 328 tiles 498 -> 504; 14 / 2 heads of 64, 21 tiles 40.5 -> 36.1, 204 tiles 147.4 -> 143.4, 276 tiles 173.4 -> 168.3,
// 532 tiles the same.
void mark_short_calls(prefix_attn_plan_t& p) {
  p.short_call = false;
  const int most = p.desc.head_dim == 128 ? 128 : 256;
  const bool no_prefix = p.desc.prefix_len == 0;
  const std::vector<WorkItem>& v = !p.range_items.empty() ? p.range_items : no_prefix ? p.items[1] : p.sweep_items;
  if (p.desc.dtype != PA_BF16 || v.empty() || (int64_t)v.size() > (int64_t)most * p.num_cu) return;
  int64_t items = 0, longest = 0;
  for (const WorkItem& it : v) {
    if (it.g < 0) continue;
    ++items;
    longest = std::max<int64_t>(longest, (it.nkeys + pa::KEYS_PER_TILE - 1) / pa::KEYS_PER_TILE + (it.pkeys + pa::KEYS_PER_TILE - 1) / pa::KEYS_PER_TILE);
  }
  p.short_call = (items + p.num_cu - 1) / p.num_cu * longest <= most;
}

// Backward, dK/dV pass: one item per block of KEYS_PER_KEY_ITEM keys of a kv head.  A prefix
// block streams the stacked rows of every rollout, all blocks of a kv head in the same order,
// so (as in the prefix pass) one kv head's blocks are kept on a fixed subset of XCDs and share
// the streamed Q/dO tiles through that subset's L2.  A suffix block streams the rollout's rows
// from its first key on; longest first.
void build_key_items(prefix_attn_plan_t& p) {
  const int Hkv = p.desc.num_kv_heads;
  const int P = (int)p.desc.prefix_len;
  const int KB = pa::KEYS_PER_KEY_ITEM;
  std::vector<pa::KeyItem>& pre = p.key_items[0];
  pre.clear();
  p.row_splits = 1;
  if (P > 0) {
    // One workgroup per CU runs at a time and all items of a launch take equally long, so the launch
    // takes ceil(items / CUs) rounds.  Few key blocks (a short prefix) leave CUs idle, and a count
    // just above a multiple of the CU count pays a whole round for its tail.  Splitting the streamed
    // rows over R items per key block shortens the rounds; it costs a prologue/epilogue per item
    // (about 3 tile steps) and, for R > 1, writing and re-reading fp32 partials (about 0.03 tile
    // steps per item).  Take the R that minimises this estimate; keep R = 1 unless it gains 2 %.
    const int64_t row_tiles = p.Mpad / pa::ROWS_PER_ROW_TILE;
    const int64_t blocks = (int64_t)Hkv * ((P + KB - 1) / KB);
    auto cost = [&](int64_t r) {
      const int64_t rounds = (blocks * r + p.num_cu - 1) / p.num_cu;
      return (double)rounds * ((double)((row_tiles + r - 1) / r) + 3.0) + (r > 1 ? 0.03 * (double)(blocks * r) : 0.0);
    };
    int64_t R = 1;
    double best = 0.98 * cost(1);
    for (int64_t r = 2; r <= 16 && row_tiles / r >= 64; ++r)
      if (cost(r) < best) {
        best = cost(r);
        R = r;
      }
    p.row_splits = (int32_t)R;
    const int64_t per_split = (row_tiles + R - 1) / R;
    std::vector<std::vector<pa::KeyItem>> per_head(Hkv);
    for (int c = 0; c < Hkv; ++c)
      for (int key0 = 0; key0 < P; key0 += KB)
        for (int r = 0; r < (int)R; ++r) {
          const int32_t t0 = (int32_t)std::min<int64_t>(r * per_split, row_tiles);
          const int32_t t1 = (int32_t)std::min<int64_t>((r + 1) * per_split, row_tiles);
          per_head[c].push_back({-1, key0, c, std::min(KB, P - key0), t0, t1, r, 0});
        }
    interleave_over_xcds(per_head, p.num_xcd, pa::KeyItem{-1, 0, -1, 0, 0, 0, 0, 0}, pre);
  }
  // A rollout's own key blocks.  Row r (position i) sees key j of its rollout iff i >= j, so a block of keys
  // [key0, key0 + n) needs the mask only on the rows at positions key0 .. key0 + n - 2 (the diagonal) and in
  // the rollout's last row tile when that tile also holds rows of the next rollout; every tile between is
  // fully visible.  Long rollouts (bf16) therefore run as two items per block: the masked kernel on the
  // diagonal tiles plus that last tile, the mask-free kernel on the tiles between, each leaving fp32 partial
  // gradients that a reduction adds.  The mask-free items walk their tiles from the rollout's end backwards:
  // all blocks of a rollout share that end, so the blocks running at the same time stream the same Q/dO tiles
  // and share them in L2, where the masked kernel, which starts every block at its own diagonal, fetched
  // 40 GB per launch for a 32,768-token sequence.  Short rollouts keep one masked item per block.
  std::vector<pa::KeyItem>& suf = p.key_items[1];
  std::vector<pa::KeyItem>& full = p.key_items_full;
  suf.clear();
  full.clear();
  const int RT = pa::ROWS_PER_ROW_TILE;
  struct Ranges { int32_t tile_b, tile_full, tile_e_full, tile_e; };
  auto ranges = [&](int g, int key0, int n) {
    const int64_t m_begin = (int64_t)(p.cu[g] + key0) * p.group;
    const int64_t m_full = (int64_t)(p.cu[g] + key0 + n - 1) * p.group;  // first row that sees the whole block
    const int64_t m_end = (int64_t)p.cu[g + 1] * p.group;
    return Ranges{(int32_t)(m_begin / RT), (int32_t)((m_full + RT - 1) / RT), (int32_t)(m_end / RT),
                  (int32_t)((m_end + RT - 1) / RT)};
  };
  // Worth it for long rollouts only (measured: a 32,768-token sequence -4 ... -9 % on the pass depending on the
  // box, a 230,400-token one -6.7 %, 2,304-token rollouts +8 %: two launches, partials and a reduction for little
  // mask-free work).
  constexpr int SPLIT_MIN_TILES = 512;
  p.suffix_split = false;
  if (p.desc.dtype == PA_BF16)
    for (int g = 0; g < p.desc.num_rollouts && !p.suffix_split; ++g) {
      const Ranges r = ranges(g, 0, std::min(KB, p.lens[g]));
      p.suffix_split = r.tile_e_full - r.tile_full >= SPLIT_MIN_TILES;  // a rollout's first block has the longest mask-free range
    }
  for (int c = 0; c < Hkv; ++c)
    for (int g = 0; g < p.desc.num_rollouts; ++g)
      for (int key0 = 0; key0 < p.lens[g]; key0 += KB) {
        const int n = std::min(KB, p.lens[g] - key0);
        const Ranges r = ranges(g, key0, n);
        if (p.suffix_split && r.tile_e_full > r.tile_full) {
          suf.push_back({g, key0, c, n, r.tile_b, r.tile_full, 0, r.tile_e_full < r.tile_e ? r.tile_e_full : -1});
          // the mask-free kernel indexes keys over all packed tokens: key0 is the packed token index here
          full.push_back({-2, p.cu[g] + key0, c, n, r.tile_full, r.tile_e_full, g, -1});
        } else {
          suf.push_back({g, key0, c, n, r.tile_b, r.tile_e, 0, -1});
          if (p.suffix_split) full.push_back({-1, p.cu[g] + key0, c, n, 0, 0, g, -1});  // no tiles
        }
      }
  auto tiles_of = [](const pa::KeyItem& a) { return a.tile1 - a.tile0 + (a.extra_tile >= 0 ? 1 : 0); };
  std::stable_sort(suf.begin(), suf.end(), [&](const pa::KeyItem& a, const pa::KeyItem& b) { return tiles_of(a) > tiles_of(b); });
  std::stable_sort(full.begin(), full.end(), [&](const pa::KeyItem& a, const pa::KeyItem& b) { return tiles_of(a) > tiles_of(b); });
  if (!full.empty()) {  // one kv head per subset of XCDs, longest first inside a head (-1.3 % on the pass)
    std::vector<std::vector<pa::KeyItem>> per_head(Hkv);
    for (const pa::KeyItem& it : full) per_head[it.c].push_back(it);
    interleave_over_xcds(per_head, p.num_xcd, pa::KeyItem{-1, 0, -1, 0, 0, 0, 0, -1}, full);
  }
}

// The launch list of the bf16 dK/dV pass.  With fewer than four items per CU, prefix blocks, mask-free and masked own
// blocks run in one launch, longest items first, so that the last round of one kind is filled with items of another:
// 5,377 prefix keys, 5 rollouts of 37 ... 1,901 tokens, 14 / 2 heads of 64: 131 + 199 us in two launches, 155 in one
// (own blocks cut, see below); 4,096 prefix keys, 8 rollouts of 1,152, 28 / 4 heads of 128: the whole backward pass 1 %
// faster (2,090 -> 2,067 us in alternating calls).  Larger launches lose nothing to their last round, and the kernel that
// holds both kinds runs the mask-free items 1 % slower (32,768 own keys: 13.44 ms in two launches, 13.52 in one), so they
// stay two launches.
//
// A launch with fewer than two items per CU is as long as its longest item, and that is often an own block (the first
// keys of a rollout are seen by all of its rows).  Those blocks are then cut into ranges of at most `limit` row
// tiles, each leaving a partial; the limit is the one for which list scheduling over the CUs ends first, the time of the
// partials (written and read at 4 TB/s, and the launch that adds them) included.  Time of a row tile: 1.87 (1.0) us at
// D = 128 (64).  Backward pass with 2 ... 16 ranges a block: 4 heads of 128, 9,115 tokens 402 us whole, 352 (2 ranges,
// taken), 373 (16); 28 / 4 heads, 2,600 tokens 565 whole, 240 (5, taken), 265 (16); 4,096 prefix keys, 2 x 1,250 tokens 746
// whole, 590 (5, taken).  Launches with more items keep whole blocks: their partials would be re-read for a tail that is
// short anyway.
void build_key_launch(prefix_attn_plan_t& p) {
  p.key_launch.clear();
  p.key_sums.clear();
  p.key_slots = 0;
  if (p.desc.dtype != PA_BF16) return;
  const pa::KeyItem pad{-1, 0, -1, 0, 0, 0, -1, -1};
  const bool cut_prefix = p.row_splits > 1;
  auto tiles_of = [](const pa::KeyItem& a) { return a.tile1 - a.tile0 + (a.extra_tile >= 0 ? 1 : 0); };

  size_t prefix_real = 0;
  int prefix_tiles = 0;
  for (const pa::KeyItem& it : p.key_items[0])
    if (it.c >= 0) {
      ++prefix_real;
      prefix_tiles = std::max(prefix_tiles, it.tile1 - it.tile0);
    }
  int limit = 0;  // most row tiles of an own item; 0: no limit
  if (!p.suffix_split && !p.key_items[1].empty() && prefix_real + p.key_items[1].size() < 2 * (size_t)p.num_cu) {
    const double tile_us = p.desc.head_dim == 128 ? 1.87 : 1.0;
    const double slot_us = 2.0 * pa::KEYS_PER_KEY_ITEM * p.desc.head_dim * 4 * 2 / 4e6, launch_us = 5.0;
    const int longest = tiles_of(p.key_items[1].front());
    std::vector<int> cost;  // half tiles
    double whole = 1e30, best = 1e30;
    for (int n = 1; n <= 16 && (n == 1 || longest / n >= 16); n += 1 + n / 6) {
      const int lim = (longest + n - 1) / n;
      size_t slots = 0;
      cost.clear();
      for (const pa::KeyItem& it : p.key_items[0])
        if (it.c >= 0) cost.push_back(2 * (it.tile1 - it.tile0) + 6);
      for (const pa::KeyItem& it : p.key_items[1]) {
        const int t = tiles_of(it), k = n == 1 ? 1 : (t + lim - 1) / lim;
        if (k > 1) slots += k;
        for (int i = 0; i < k; ++i) cost.push_back(2 * t / k + (k > 1 ? 7 : 6));
      }
      if (slots > 4 * (size_t)p.num_cu) continue;  // at most 128 (64) MiB of workspace; the best cuts above have 100 to 570
      const double extra = slots ? slots * slot_us + launch_us : 0.0;
      const double enough = std::min(whole, 1.02 * best);  // of two that are within 2 % the one with shorter items
      const double us = list_schedule(cost, p.num_cu, 2.0 * (enough - extra) / tile_us) / 2.0 * tile_us + extra;
      if (n == 1) whole = best = 0.95 * us;
      else if (us < enough) {
        best = std::min(best, us);
        limit = lim;
      }
    }
  }

  // slots: those of a block are adjacent, in the order in which the reduction adds them
  std::vector<int> first;  // of a prefix block
  const int prefix_blocks = (int)((p.desc.prefix_len + pa::KEYS_PER_KEY_ITEM - 1) / pa::KEYS_PER_KEY_ITEM);
  if (cut_prefix) {
    first.assign((size_t)p.desc.num_kv_heads * prefix_blocks, -1);
    for (const pa::KeyItem& it : p.key_items[0]) {
      if (it.c < 0) continue;
      int& slot0 = first[(size_t)it.c * prefix_blocks + it.key0 / pa::KEYS_PER_KEY_ITEM];
      if (slot0 >= 0) continue;
      slot0 = p.key_slots;
      p.key_slots += p.row_splits;
      p.key_sums.push_back({0, it.key0, it.c, it.nkeys, slot0, p.row_splits});
    }
  }
  std::vector<pa::KeyItem> own;
  // split pass: where the masked item of a block stands in `own`.  Blocks of a kv head are numbered cu[g] / KB + g + key0 / KB
  // (unique: a rollout leaves at most one number unused)
  const int KB = pa::KEYS_PER_KEY_ITEM;
  const int64_t numbers = p.T / KB + p.desc.num_rollouts;
  std::vector<int> masked(p.suffix_split ? numbers * p.desc.num_kv_heads : 0);
  auto number = [&](int c, int g, int key0) { return c * numbers + p.cu[g] / KB + g + key0 / KB; };
  own.reserve(p.key_items[1].size());
  for (pa::KeyItem it : p.key_items[1]) {
    const int t = tiles_of(it), n = limit ? (t + limit - 1) / limit : 1;
    const int packed = p.cu[it.g] + it.key0;
    it.slot = -1;
    if (it.extra_tile >= 0 || n == 1) {
      if (p.suffix_split) masked[number(it.c, it.g, it.key0)] = (int)own.size();
      own.push_back(it);
      continue;
    }
    p.key_sums.push_back({1, packed, it.c, it.nkeys, p.key_slots, n});
    for (int i = 0; i < n; ++i) {
      pa::KeyItem part = it;
      part.tile0 = it.tile0 + (int)((int64_t)t * i / n);
      part.tile1 = it.tile0 + (int)((int64_t)t * (i + 1) / n);
      part.slot = p.key_slots++;
      own.push_back(part);
    }
  }
  std::vector<pa::KeyItem> full;
  full.reserve(p.key_items_full.size());
  for (pa::KeyItem it : p.key_items_full) {
    if (it.c >= 0 && it.tile1 > it.tile0) {  // masked item and mask-free item: one partial each
      pa::KeyItem& m = own[masked[number(it.c, it.slot, it.key0 - p.cu[it.slot])]];
      p.key_sums.push_back({1, it.key0, it.c, it.nkeys, p.key_slots, 2});
      m.slot = p.key_slots++;
      it.slot = p.key_slots++;
      full.push_back(it);
    } else {
      full.push_back(pad);  // keeps the list's layout over the XCDs
    }
  }
  std::stable_sort(own.begin(), own.end(), [&](const pa::KeyItem& a, const pa::KeyItem& b) { return tiles_of(a) > tiles_of(b); });

  // launch order; the lists laid out over the XCDs start at a multiple of the XCD count
  size_t real = own.size() + prefix_real;
  for (const pa::KeyItem& it : full) real += it.c >= 0;
  p.key_launch.reserve(full.size() + p.key_items[0].size() + own.size() + 4 * p.num_xcd);
  auto append = [&](const pa::KeyItem* b, const pa::KeyItem* e) {
    while (p.key_launch.size() % p.num_xcd != 0) p.key_launch.push_back(pad);
    p.key_launch.insert(p.key_launch.end(), b, e);
  };
  auto append_prefix = [&]() {
    append(nullptr, nullptr);
    for (pa::KeyItem it : p.key_items[0]) {
      // the prefix list's items carry their row range's number
      it.slot = it.c >= 0 && cut_prefix ? first[(size_t)it.c * prefix_blocks + it.key0 / pa::KEYS_PER_KEY_ITEM] + it.slot : -1;
      p.key_launch.push_back(it);
    }
  };
  p.key_mask_free = -1;
  append(full.data(), full.data() + full.size());
  if (real >= 4 * (size_t)p.num_cu) {
    append_prefix();
    append(nullptr, nullptr);  // pads, so that the count below is where the masked items begin
    p.key_mask_free = (int64_t)p.key_launch.size();
    append(own.data(), own.data() + own.size());
    return;
  }
  size_t long_own = 0;
  while (long_own < own.size() && full.empty() && tiles_of(own[long_own]) > prefix_tiles) ++long_own;
  append(own.data(), own.data() + long_own);
  append_prefix();
  append(own.data() + long_own, own.data() + own.size());
}

// How many 16-key or 16-row blocks an item of an fp32 backward launch may hold at most (0: no limit) so that one workgroup
// per CU ends early.  blocks: those that each whole item streams; a workgroup's 8 wavefronts take one each at a time, one such
// step lasting step_us, its start and end OVERHEAD steps.  Candidates are compared by list scheduling as in list_schedule, but
// over the few lengths that occur and not item by item: every fp32 plan pays for the search, also one that only runs forwards.
int f32_limit(const std::vector<int>& blocks, int cus, double step_us, double slot_us) {
  constexpr int OVERHEAD = 2;
  constexpr double LAUNCH_US = 6.0;  // the sums
  if (blocks.empty() || blocks.size() >= 4 * (size_t)cus) return 0;
  std::vector<std::pair<int, int>> runs;  // neighbours of equal length: {length, how many}
  for (int b : blocks)
    if (!runs.empty() && runs.back().first == b) ++runs.back().second; else runs.push_back({b, 1});
  const int longest = (std::max_element(runs.begin(), runs.end())->first + 7) / 8;
  int64_t steps = 0;                           // of all items, their starts and ends among them
  for (const auto& [b, times] : runs) steps += (int64_t)times * ((b + 7) / 8 + OVERHEAD);
  std::vector<int> of_length(longest + 1);     // items by their steps
  std::vector<std::pair<int, int>> free;       // {when, how many CUs} are free then, ascending from `head` on
  // When the last item ends, in steps, longest first on whichever CU is free; at least `enough` if that is certain.
  auto schedule = [&](double enough) {
    free.assign(1, {0, cus});
    size_t head = 0;
    int end = 0;
    for (int t = longest; t > 0; --t)
      for (int left = of_length[t]; left > 0;) {
        const int n = std::min(left, free[head].second), at = free[head].first + t + OVERHEAD;
        left -= n;
        end = std::max(end, at);
        if (end >= enough) return end;
        if ((free[head].second -= n) == 0) ++head;
        auto pos = std::lower_bound(free.begin() + head, free.end(), std::make_pair(at, 0));
        if (pos != free.end() && pos->first == at) pos->second += n; else free.insert(pos, {at, n});
      }
    return end;
  };
  int limit = 0;
  double best = 0.0;
  for (int n = 1; n <= 16 && (n == 1 || longest / n >= 2); n += 1 + n / 6) {
    const int most = 8 * ((longest + n - 1) / n);
    size_t slots = 0;
    std::fill(of_length.begin(), of_length.end(), 0);
    for (const auto& [b, times] : runs) {
      const int k = (b + most - 1) / most;
      if (k > 1) slots += (size_t)k * times;
      of_length[((b + k - 1) / k + 7) / 8] += k * times;
    }
    if (slots > 4 * (size_t)cus) break;  // more ranges would only have more
    const double extra = slots ? slots * slot_us + LAUNCH_US : 0.0;
    const double us = schedule(n == 1 ? 1e30 : (best - extra) / step_us) * step_us + extra;
    if (n == 1) {
      best = 0.95 * us;
      if ((double)steps / cus * step_us + LAUNCH_US >= best) return 0;  // nothing to gain: cuts only add steps
    } else if (us < best) {
      best = us;
      limit = most;
    }
  }
  return limit;
}

// fp32 backward launches of few blocks, cut like the bf16 ones: blocks of 16 rows into ranges of 16-key blocks (dQ), blocks
// of 16 keys into ranges of stacked rows (dK/dV), in the lists that the bf16 path uses for the same purpose (empty: whole
// blocks), with slots of 16 rows or 2 x 16 keys.  Step times measured by whole blocks of different length, at D = 128 (64): dQ
// 3.7 (2.1) us, dK/dV 4.6 ... 5.0 (2.6 ... 2.8).  8 / 2 heads of 128, 900 tokens of 4 rollouts over 1,000 prefix keys, 126 + 118
// blocks of keys: dK/dV 147 us whole, 124 / 109 / 123 / 111 / 121 in 2 ... 6 ranges (3 taken, the sums 5 us); dQ 90 us whole
// (452 blocks of rows, left so), 99 / 110 / 105 in 2 / 3 / 4.  A like call at D = 64: dK/dV and sums 82 us whole, 73 / 66 / 75 in 2 / 3 / 4
// (3 taken, 70); dQ 50 whole, 48 / 49 / 47.  The whole backward of 24 shapes of 96 ... 2,000 tokens, what the rule takes against whole
// blocks and against the kernels before rows went through LDS: D = 128 0.29 ... 1.0 and 0.24 ... 0.89, D = 64 0.33 ... 1.0 and
// 0.32 ... 0.95 of their time, none slower.  (At D = 64 two dQ workgroups fit a CU; the rule counts one and cuts too little there: 342 blocks
// of rows 48 us, 38 in two ranges each.)  Launches of four blocks a CU and more stay whole: their last round is short against the rest.
void build_f32_cuts(prefix_attn_plan_t& p) {
  if (p.desc.dtype != PA_F32) return;
  const int np = (int)((p.desc.prefix_len + 15) / 16), Hkv = p.desc.num_kv_heads;
  const bool d128 = p.desc.head_dim == 128;
  const double slot_us = 16.0 * p.desc.head_dim * 4 * 2 / 4e6;
  std::vector<int> blocks;
  blocks.reserve(4 * (size_t)p.num_cu);
  if (p.f32_blocks[1].size() < 4 * (size_t)p.num_cu)
    for (const WorkItem& it : p.f32_blocks[1])
      blocks.push_back(np + ((std::min(it.row0 + 16, p.lens[it.g] * p.group) - 1) / p.group + 16) / 16);
  if (const int limit = f32_limit(blocks, p.num_cu, d128 ? 3.75 : 2.0, slot_us)) {
    std::vector<std::pair<int, WorkItem>> items;
    for (size_t n = 0; n < blocks.size(); ++n) {
      WorkItem it = p.f32_blocks[1][n];
      const int k = (blocks[n] + limit - 1) / limit;
      if (k > 1) {
        p.dq_sums.push_back({p.cu[it.g], it.row0, it.c, std::min(16, p.lens[it.g] * p.group - it.row0), p.dq_slots, k});
        for (int i = 0; i < k; ++i) {
          it.key0 = (int)((int64_t)blocks[n] * i / k);
          it.nkeys = (int)((int64_t)blocks[n] * (i + 1) / k) - it.key0;
          it.split = p.dq_slots++;
          items.push_back({it.nkeys, it});
        }
      } else {
        it.nkeys = blocks[n];
        it.split = -1;
        items.push_back({blocks[n], it});
      }
    }
    std::stable_sort(items.begin(), items.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
    for (const auto& it : items) p.dq_launch.push_back(it.second);
  }

  blocks.clear();
  std::vector<pa::KeyItem> keys;
  if ((np + p.T / 16 + p.desc.num_rollouts) * Hkv < 4 * (int64_t)p.num_cu && (int64_t)p.T * p.group < (int64_t)1 << 30) {
    keys.reserve(4 * (size_t)p.num_cu);
    auto add = [&](int g, int n, int first_row, int end_row) {
      for (int key0 = 0; key0 < n; key0 += 16)
        for (int c = 0; c < Hkv; ++c) {
          const int row0 = first_row + (g < 0 ? 0 : key0 * p.group);
          keys.push_back({g, key0, c, std::min(16, n - key0), row0, end_row, -1, -1});
          blocks.push_back((end_row - row0 + 15) / 16);
        }
    };
    add(-1, (int)p.desc.prefix_len, 0, (int)p.T * p.group);
    for (int g = 0; g < p.desc.num_rollouts; ++g) add(g, p.lens[g], p.cu[g] * p.group, p.cu[g + 1] * p.group);
  }
  if (const int limit = f32_limit(blocks, p.num_cu, d128 ? 4.7 : 2.5, 2.0 * slot_us)) {
    for (size_t n = 0; n < blocks.size(); ++n) {
      pa::KeyItem it = keys[n];
      const int k = (blocks[n] + limit - 1) / limit, row0 = it.tile0, end = it.tile1;
      if (k > 1) p.key_sums.push_back({it.g >= 0, it.key0 + (it.g >= 0 ? p.cu[it.g] : 0), it.c, it.nkeys, p.key_slots, k});
      for (int i = 0; i < k; ++i) {
        it.tile0 = row0 + 16 * (int)((int64_t)blocks[n] * i / k);
        it.tile1 = std::min(end, row0 + 16 * (int)((int64_t)blocks[n] * (i + 1) / k));
        it.slot = k > 1 ? p.key_slots++ : -1;
        p.key_launch.push_back(it);
      }
    }
    std::stable_sort(p.key_launch.begin(), p.key_launch.end(),
                     [](const pa::KeyItem& a, const pa::KeyItem& b) { return a.tile1 - a.tile0 > b.tile1 - b.tile0; });
  }
}

// Backward workspace: delta and the re-ordered LSE (used by the fp32 path); for bf16 also the stacked Q/dO copies, the
// per-row statistics and the transposed K images.
void layout_backward_workspace(prefix_attn_plan_t& p) {
  const prefix_attn_desc_t& d = p.desc;
  const size_t rows = (size_t)p.T * d.num_q_heads;
  p.Mpad = ((int64_t)p.T * p.group + pa::ROWS_PER_ROW_TILE - 1) / pa::ROWS_PER_ROW_TILE * pa::ROWS_PER_ROW_TILE;
  p.boff_delta = 0;
  p.boff_lse_th = align_up(rows * sizeof(float), 256);
  size_t end = 2 * p.boff_lse_th;
  if (d.dtype == PA_BF16) {
    const size_t stacked = align_up((size_t)d.num_kv_heads * p.Mpad * d.head_dim * 2, 256);
    const size_t stats = align_up((size_t)d.num_kv_heads * p.Mpad * 4, 256);
    const size_t image = (size_t)d.head_dim * pa::KEYS_PER_TILE * 2;
    p.boff_qs = end;
    p.boff_dos = p.boff_qs + stacked;
    p.boff_lse2s = p.boff_dos + stacked;
    p.boff_deltas = p.boff_lse2s + stats;
    p.boff_toks = p.boff_deltas + stats;
    p.boff_ktp = p.boff_toks + stats;
    p.boff_kts = p.boff_ktp + align_up((size_t)d.num_kv_heads * p.tiles_prefix * image, 256);
    end = p.boff_kts + align_up((size_t)d.num_kv_heads * p.tiles_suffix * image, 256);
    p.boff_part = end;  // fp32 partial dK, dV: [key_slots][2][KEYS_PER_KEY_ITEM][D]
    end += align_up((size_t)p.key_slots * 2 * pa::KEYS_PER_KEY_ITEM * d.head_dim * sizeof(float), 256);
    p.boff_dqpart = end;  // fp32 partial dQ: [dq_slots][ROWS_PER_ITEM][D]
    end += align_up((size_t)p.dq_slots * pa::ROWS_PER_ITEM * d.head_dim * sizeof(float), 256);
  } else {  // partial sums of cut blocks: [key_slots][2][16][D], [dq_slots][16][D]
    p.boff_part = end;
    p.boff_dqpart = p.boff_part + (size_t)p.key_slots * 2 * 16 * d.head_dim * sizeof(float);
    end = p.boff_dqpart + (size_t)p.dq_slots * 16 * d.head_dim * sizeof(float);
  }
  p.bws_bytes = end;
}

}  // namespace

extern "C" {

int prefix_attn_plan(const prefix_attn_desc_t* desc, prefix_attn_plan_t** plan_out, size_t* workspace_bytes_out) {
  if (plan_out) *plan_out = nullptr;
  if (!desc || !plan_out || !workspace_bytes_out) return PA_ERR_NULL;
  const int st = validate(desc);
  if (st != PA_OK) return st;
  prefix_attn_plan_t* p = new (std::nothrow) prefix_attn_plan_t();
  if (!p) return PA_ERR_ALLOC;
  if (desc->device >= 0) {  // size the schedule for the device it will run on
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, desc->device) != hipSuccess || cus < 1) {
      (void)hipGetLastError();
      delete p;
      return PA_ERR_HIP;
    }
    if (cus != pa::NUM_CU) {  // not the layout the XCD interleaving is built for
      p->num_cu = cus;
      p->num_xcd = 1;
    }
  }
  try {
    p->desc = *desc;
    p->lens.assign(desc->suffix_lens, desc->suffix_lens + desc->num_rollouts);
    p->desc.suffix_lens = p->lens.data();
    p->cu.assign(desc->num_rollouts + 1, 0);
    for (int g = 0; g < desc->num_rollouts; ++g) p->cu[g + 1] = p->cu[g] + p->lens[g];
    p->T = p->cu.back();
    p->vt_off.assign(desc->num_rollouts + 1, 0);
    for (int g = 0; g < desc->num_rollouts; ++g)
      p->vt_off[g + 1] = p->vt_off[g] + (p->lens[g] + pa::KEYS_PER_TILE - 1) / pa::KEYS_PER_TILE;
    p->tiles_suffix = p->vt_off.back();
    p->tiles_prefix = (int32_t)((desc->prefix_len + pa::KEYS_PER_TILE - 1) / pa::KEYS_PER_TILE);
    p->group = desc->num_q_heads / desc->num_kv_heads;
    build_prefix_items(*p);
    build_suffix_items(*p);
    build_f32_blocks(*p);
    build_dq_items(*p);
    build_sweep_items(*p);
    p->Mpad = ((int64_t)p->T * p->group + pa::ROWS_PER_ROW_TILE - 1) / pa::ROWS_PER_ROW_TILE * pa::ROWS_PER_ROW_TILE;
    build_key_items(*p);
    build_key_launch(*p);
    build_dq_launch(*p);
    build_f32_cuts(*p);
  } catch (const std::bad_alloc&) {
    delete p;
    return PA_ERR_ALLOC;
  }
  const size_t rows = (size_t)p->T * desc->num_q_heads;
  const size_t o_bytes = align_up(rows * desc->head_dim * sizeof(float), 256);
  const size_t l_bytes = align_up(rows * sizeof(float), 256);
  const size_t ks = (size_t)p->key_splits;  // the prefix pass leaves one partial per key split, the suffix pass one more
  try {
    const size_t tiles = (size_t)p->tiles_prefix + p->tiles_suffix;
    const size_t items = std::max({p->items[0].size(), p->items[1].size(), p->sweep_items.size()});
    build_range_items(*p, l_bytes + desc->num_kv_heads * tiles * desc->head_dim * pa::KEYS_PER_TILE * 2 +
                              items * pa::WAVES_PER_ITEM * sizeof(int32_t) + 4 * 256,
                      o_bytes + l_bytes);
    mark_short_calls(*p);
  } catch (const std::bad_alloc&) {
    delete p;
    return PA_ERR_ALLOC;
  }
  p->off_o1 = 0;
  p->off_o2 = ks * o_bytes;
  p->off_lse1 = (ks + 1) * o_bytes;
  p->off_lse2 = p->off_lse1 + ks * l_bytes;
  // the range list's slots lie over the partials of the passes, which a call that uses it does not run
  const size_t slot_rows = (size_t)p->range_slots * pa::ROWS_PER_ITEM;
  p->off_slot_lse = align_up(slot_rows * desc->head_dim * sizeof(float), 256);
  p->off_lse = std::max(p->off_lse1 + (ks + 1) * l_bytes, p->off_slot_lse + align_up(slot_rows * sizeof(float), 256));
  p->off_vtp = p->off_lse + l_bytes;
  size_t end = p->off_vtp;
  if (desc->dtype == PA_BF16) {  // transposed-V tile images, bf16 path only
    const size_t image = (size_t)desc->head_dim * pa::KEYS_PER_TILE * 2;
    p->off_vts = p->off_vtp + align_up((size_t)desc->num_kv_heads * p->tiles_prefix * image, 256);
    end = p->off_vts + align_up((size_t)desc->num_kv_heads * p->tiles_suffix * image, 256);
    // one word per (work item, wavefront) of the longest work list: a pass's common kernel tells its careful
    // kernel which items to redo; the passes run one after the other and share the region
    const size_t items = std::max({p->items[0].size(), p->items[1].size(), p->sweep_items.size(), p->range_items.size()});
    p->off_flags = end;
    end += align_up(items * pa::WAVES_PER_ITEM * sizeof(int32_t), 256);
  }
  p->ws_bytes = end;
  layout_backward_workspace(*p);

  if (desc->device >= 0) {
    int prev = 0;
    bool ok = hipGetDevice(&prev) == hipSuccess && hipSetDevice(desc->device) == hipSuccess;
    if (ok) {
      // every list of the plan in one allocation and one copy (seven of each were a third of a plan's time)
      std::vector<std::pair<void**, std::pair<const void*, size_t>>> lists;
      size_t total = 0;
      auto add = [&](auto** dst, const auto& v) {
        if (v.empty()) return;
        lists.push_back({(void**)dst, {v.data(), v.size() * sizeof(v[0])}});
        total += align_up(v.size() * sizeof(v[0]), 256);
      };
      try {
        add(&p->d_cu, p->cu);
        add(&p->d_vt_off, p->vt_off);
        if (desc->dtype != PA_F32) {  // fp32: one sweep over its own blocks of rows
          add(&p->d_items[0], p->items[0]);
          add(&p->d_items[1], p->items[1]);
        }
        for (int s = 0; s < 2; ++s) add(&p->d_f32_blocks[s], p->f32_blocks[s]);
        add(&p->d_sweep_items, p->sweep_items);
        add(&p->d_range_items, p->range_items);
        add(&p->d_range_sums, p->range_sums);
        add(&p->d_dq_launch, p->dq_launch);
        add(&p->d_dq_sums, p->dq_sums);
        add(&p->d_key_launch, p->key_launch);
        add(&p->d_key_sums, p->key_sums);
        std::vector<char> host(total);
        ok = hipMalloc(&p->d_lists, total) == hipSuccess;
        size_t at = 0;
        for (const auto& [dst, src] : lists) {
          std::copy_n(static_cast<const char*>(src.first), src.second, host.data() + at);
          *dst = static_cast<char*>(p->d_lists) + at;
          at += align_up(src.second, 256);
        }
        ok = ok && hipMemcpy(p->d_lists, host.data(), total, hipMemcpyHostToDevice) == hipSuccess;
      } catch (const std::bad_alloc&) {
        ok = false;
      }
      // set-up for prefix_attn_forward_static: look its workspace up now, with the plan's device current,
      // so that the call itself only reads a table
      void* unused = nullptr;
      ok = ok && pa::static_scratch(desc->device, &unused) == PA_OK;
      (void)hipSetDevice(prev);
    }
    if (!ok) {
      (void)hipGetLastError();
      prefix_attn_destroy(p);
      return PA_ERR_ALLOC;
    }
  }
  *plan_out = p;
  *workspace_bytes_out = p->ws_bytes;
  return PA_OK;
}

void prefix_attn_destroy(prefix_attn_plan_t* plan) {
  if (!plan) return;
  if (plan->d_lists) (void)hipFree(plan->d_lists);
  delete plan;
}

const char* prefix_attn_status_string(int status) {
  switch (status) {
    case PA_OK: return "ok";
    case PA_ERR_NULL: return "a required pointer is NULL";
    case PA_ERR_SHAPE: return "a size is out of range or inconsistent";
    case PA_ERR_UNSUPPORTED: return "valid but unsupported configuration";
    case PA_ERR_ALIGN: return "a device pointer is not 16-byte aligned";
    case PA_ERR_WORKSPACE: return "workspace too small";
    case PA_ERR_ALLOC: return "allocation failed";
    case PA_ERR_HIP: return "HIP runtime call or kernel launch failed";
    default: return "unknown status";
  }
}

int prefix_attn_plan_tiles(const prefix_attn_plan_t* plan, int32_t* rows_per_item, int32_t* keys_per_tile) {
  if (!plan || !rows_per_item || !keys_per_tile) return PA_ERR_NULL;
  *rows_per_item = pa::ROWS_PER_ITEM;
  *keys_per_tile = pa::KEYS_PER_TILE;
  return PA_OK;
}

int64_t prefix_attn_plan_num_items(const prefix_attn_plan_t* plan, int32_t pass) {
  if (!plan || pass < 0 || pass > 3) return -1;
  return (int64_t)(pass == 3 ? plan->sweep_items : pass == 2 ? plan->dq_items : plan->items[pass]).size();
}

int prefix_attn_plan_items(const prefix_attn_plan_t* plan, int32_t pass, int32_t* items_out) {
  if (!plan || !items_out) return PA_ERR_NULL;
  if (pass < 0 || pass > 3) return PA_ERR_SHAPE;
  const std::vector<WorkItem>& v = pass == 3 ? plan->sweep_items : pass == 2 ? plan->dq_items : plan->items[pass];
  for (size_t n = 0; n < v.size(); ++n) {
    items_out[6 * n + 0] = v[n].g;
    items_out[6 * n + 1] = v[n].row0;
    items_out[6 * n + 2] = v[n].c;
    items_out[6 * n + 3] = v[n].nkeys;
    items_out[6 * n + 4] = v[n].key0;
    items_out[6 * n + 5] = v[n].pkeys;
  }
  return PA_OK;
}

namespace {

// What a launch list consists of; a list that the plan's data type does not have is empty.  (The plan keeps the cut launches of
// a backward, lists 1 and 2 in bf16 and 6 and 7 in fp32, in the same members.)
struct LaunchList {
  bool exists = false, summed = false;  // summed: its cut blocks leave partial results in slots
  const std::vector<WorkItem>* rows = nullptr;
  const std::vector<pa::KeyItem>* keys = nullptr;
  const std::vector<pa::RangeSum>* row_sums = nullptr;
  const std::vector<pa::KeySum>* key_sums = nullptr;
  int64_t slots = 0;
  int rows_per_block = 0, waves = 0;  // lists of whole fp32 blocks
};

LaunchList launch_list(const prefix_attn_plan_t* plan, int32_t list) {
  LaunchList l;
  if (!plan) return l;
  const bool f32 = plan->desc.dtype == PA_F32;
  auto rows = [&](bool here, const std::vector<WorkItem>& items, const std::vector<pa::RangeSum>& sums, int32_t slots) {
    l.summed = true;
    if (here) {
      l.rows = &items;
      l.row_sums = &sums;
      l.slots = slots;
    }
  };
  auto keys = [&](bool here) {
    l.summed = true;
    if (here) {
      l.keys = &plan->key_launch;
      l.key_sums = &plan->key_sums;
      l.slots = plan->key_slots;
    }
  };
  auto whole = [&](int which, int rows_per_block, int waves) {
    if (!f32) return;
    l.rows = &plan->f32_blocks[which];
    l.rows_per_block = rows_per_block;
    l.waves = waves;
  };
  l.exists = true;
  switch (list) {
    case 0: rows(!f32, plan->range_items, plan->range_sums, plan->range_slots); break;
    case 1: rows(!f32, plan->dq_launch, plan->dq_sums, plan->dq_slots); break;
    case 2: keys(!f32); break;
    case 3: whole(0, plan->f32_rows, plan->f32_waves); break;
    case 4: whole(1, 16, 8); break;
    case 6: rows(f32, plan->dq_launch, plan->dq_sums, plan->dq_slots); break;
    case 7: keys(f32); break;
    default: l.exists = false;
  }
  return l;
}

}  // namespace

int64_t prefix_attn_plan_num_launch_items(const prefix_attn_plan_t* plan, int32_t list) {
  const LaunchList l = launch_list(plan, list);
  if (!l.exists) return -1;
  return (int64_t)(l.keys ? l.keys->size() : l.rows ? l.rows->size() : 0);
}

int prefix_attn_plan_launch_items(const prefix_attn_plan_t* plan, int32_t list, int32_t* items_out) {
  if (!plan || !items_out) return PA_ERR_NULL;
  const LaunchList l = launch_list(plan, list);
  if (!l.exists) return PA_ERR_SHAPE;
  auto put = [&](std::initializer_list<int32_t> v) { items_out = std::copy(v.begin(), v.end(), items_out); };
  if (l.keys)
    for (const pa::KeyItem& it : *l.keys) put({it.g, it.key0, it.c, it.nkeys, it.tile0, it.tile1, it.extra_tile, it.slot});
  if (l.rows)
    for (const WorkItem& it : *l.rows) {
      if (l.waves) put({it.g, it.row0, it.c, l.rows_per_block, l.waves, 0, 0, -1});
      else put({it.g, it.row0, it.c, it.nkeys, it.key0, it.pkeys, it.okey0, it.split});
    }
  return PA_OK;
}

int64_t prefix_attn_plan_num_launch_sums(const prefix_attn_plan_t* plan, int32_t list) {
  const LaunchList l = launch_list(plan, list);
  if (!l.summed) return -1;
  return (int64_t)(l.key_sums ? l.key_sums->size() : l.row_sums ? l.row_sums->size() : 0);
}

int prefix_attn_plan_launch_sums(const prefix_attn_plan_t* plan, int32_t list, int32_t* sums_out) {
  if (!plan || !sums_out) return PA_ERR_NULL;
  const LaunchList l = launch_list(plan, list);
  if (!l.summed) return PA_ERR_SHAPE;
  auto put = [&](std::initializer_list<int32_t> v) { sums_out = std::copy(v.begin(), v.end(), sums_out); };
  if (l.key_sums)
    for (const pa::KeySum& s : *l.key_sums) put({s.own, s.key0, s.c, s.nkeys, s.slot0, s.nslots});
  if (l.row_sums)
    for (const pa::RangeSum& s : *l.row_sums) put({s.off_g, s.row0, s.c, s.nrows, s.slot0, s.nslots});
  return PA_OK;
}

int64_t prefix_attn_plan_launch_slots(const prefix_attn_plan_t* plan, int32_t list) {
  const LaunchList l = launch_list(plan, list);
  return l.summed ? l.slots : -1;
}

int64_t prefix_attn_plan_mask_free_items(const prefix_attn_plan_t* plan) { return plan ? plan->key_mask_free : -1; }

int prefix_attn_plan_short_call(const prefix_attn_plan_t* plan) { return plan ? plan->short_call : -1; }

int64_t prefix_attn_plan_total_tokens(const prefix_attn_plan_t* plan) { return plan ? plan->T : -1; }

int prefix_attn_backward_workspace(const prefix_attn_plan_t* plan, size_t* workspace_bytes_out) {
  if (!plan || !workspace_bytes_out) return PA_ERR_NULL;
  *workspace_bytes_out = plan->bws_bytes;
  return PA_OK;
}

int64_t prefix_attn_plan_num_key_items(const prefix_attn_plan_t* plan, int32_t pass) {
  if (!plan || pass < 0 || pass > 2) return -1;
  return (int64_t)(pass == 2 ? plan->key_items_full : plan->key_items[pass]).size();
}

int prefix_attn_plan_key_items(const prefix_attn_plan_t* plan, int32_t pass, int32_t* items_out) {
  if (!plan || !items_out) return PA_ERR_NULL;
  if (pass < 0 || pass > 2) return PA_ERR_SHAPE;
  const std::vector<pa::KeyItem>& v = pass == 2 ? plan->key_items_full : plan->key_items[pass];
  for (size_t n = 0; n < v.size(); ++n) {
    items_out[6 * n + 0] = v[n].g;
    items_out[6 * n + 1] = v[n].key0;
    items_out[6 * n + 2] = v[n].c;
    items_out[6 * n + 3] = v[n].nkeys;
    items_out[6 * n + 4] = v[n].tile0;
    items_out[6 * n + 5] = v[n].tile1;
  }
  return PA_OK;
}

int prefix_attn_plan_key_item_extra_tiles(const prefix_attn_plan_t* plan, int32_t pass, int32_t* tiles_out) {
  if (!plan || !tiles_out) return PA_ERR_NULL;
  if (pass < 0 || pass > 2) return PA_ERR_SHAPE;
  const std::vector<pa::KeyItem>& v = pass == 2 ? plan->key_items_full : plan->key_items[pass];
  for (size_t n = 0; n < v.size(); ++n) tiles_out[n] = pass == 1 ? v[n].extra_tile : -1;
  return PA_OK;
}

}  // extern "C"
