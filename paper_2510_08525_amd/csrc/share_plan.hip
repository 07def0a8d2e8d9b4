// Host side of the work list: where the end-to-end sequence of scheduling units is cut into one
// contiguous share per workgroup.  Runs on the host from the library's mirror of the lengths; the
// records are then read out of pinned memory by a small kernel (4 us, no copy engine).
//
// Cost model (paper Sec. 4.3: the residual cost of a compressed head is its sW/L tokens, so a
// share's cost is what it reads plus what it restarts): kRoundCost per round of tiles plus
// kPairStartCost for every pair that starts in the share - the load pipeline restarts on a new
// store, Q is loaded, a merge and an output or partial write follow; about 1.5 rounds by
// per-workgroup timestamps.  A pair that continues from the previous workgroup pays no start.
// The plan is the in-order greedy deal at the smallest capacity that needs no more workgroups than
// the grid has; greedy is optimal for a contiguous partition once the capacity is fixed.
#include <algorithm>
#include <cmath>
#include <vector>

#include "prefill_deal.h"
#include "rlkv_internal.h"

namespace rlkv {

// Deals the rounds out at capacity `cap`; returns the number of workgroups used.  With wg_begin /
// seg_first / seg_count non-null also records the shares.
static int deal_rounds(const int32_t* rounds, int n_pairs, int cap, int32_t* wg_begin, int32_t* seg_first,
                       int32_t* seg_count, bool single = false) {
  const int per_fresh = single ? 1 : cap / kRoundCost;     // rounds a workgroup takes of a pair it does not start
  int w = 0, used = 0, us = 0;                             // us: first unit of the pair in the end-to-end numbering
  for (int p = 0; p < n_pairs; ++p) {
    const int r = rounds[p];
    if (seg_first) { seg_first[p] = 0; seg_count[p] = 0; }
    if (r == 0) continue;                                  // inactive slot
    if (used > 0 && cap - used < kPairStartCost + kRoundCost) {
      ++w;
      used = 0;
      if (wg_begin) wg_begin[w] = us;
    }
    if (seg_first) seg_first[p] = w;
    used += kPairStartCost;
    int take = (cap - used) / kRoundCost;
    if (take > r) take = r;
    used += take * kRoundCost;
    const int rest = r - take;
    if (rest > 0) {
      const int more = (rest + per_fresh - 1) / per_fresh;          // further workgroups, the last one partly filled
      if (wg_begin)
        for (int k = 0; k < more; ++k) wg_begin[w + 1 + k] = us + kPairOverheadUnits + take + k * per_fresh;
      w += more;
      used = (rest - (more - 1) * per_fresh) * kRoundCost;
    }
    if (seg_count) seg_count[p] = w - seg_first[p] + 1;
    us += r + kPairOverheadUnits;
  }
  return w + 1;
}

int plan_shares(const int32_t* rounds, int n_pairs, int n_wg, int32_t* wg_begin, int32_t* seg_first,
                int32_t* seg_count, bool singly) {
  int64_t cost = 0, units = 0, all_rounds = 0;
  int longest = 0;
  for (int p = 0; p < n_pairs; ++p)
    if (rounds[p] > 0) {
      cost += (int64_t)rounds[p] * kRoundCost + kPairStartCost;
      units += rounds[p] + kPairOverheadUnits;
      all_rounds += rounds[p];
      if (rounds[p] > longest) longest = rounds[p];
    }
  for (int w = 0; w <= n_wg; ++w) wg_begin[w] = (int32_t)units;      // workgroups the deal does not reach stay empty
  wg_begin[0] = 0;
  if (units == 0) {
    for (int p = 0; p < n_pairs; ++p) seg_first[p] = seg_count[p] = 0;
    return 0;
  }
  // A list that the grid takes at one round per workgroup: the shortest chain of latencies there is, as long as a pair has few
  // partials (16).
  if (singly || (all_rounds <= n_wg && longest <= 16))
    return deal_rounds(rounds, n_pairs, kPairStartCost + kRoundCost, wg_begin, seg_first, seg_count, true);
  // feasible for sure: the whole list in one workgroup; look upward from the average
  int64_t cap = (cost + n_wg - 1) / n_wg;
  if (cap < kPairStartCost + kRoundCost) cap = kPairStartCost + kRoundCost;
  while (deal_rounds(rounds, n_pairs, (int)cap, nullptr, nullptr, nullptr) > n_wg) {
    // the average is nearly always within a few steps of the answer; widen the stride if not
    const int64_t step = cap / 64 > 0 ? cap / 64 : 1;
    int64_t probe = cap + step;
    if (step > 1 && deal_rounds(rounds, n_pairs, (int)probe, nullptr, nullptr, nullptr) <= n_wg) {
      // overshot: walk the last stride one by one
      ++cap;
      while (deal_rounds(rounds, n_pairs, (int)cap, nullptr, nullptr, nullptr) > n_wg) ++cap;
      break;
    }
    cap = probe;
  }
  return deal_rounds(rounds, n_pairs, (int)cap, wg_begin, seg_first, seg_count);
}

void plan_whole_pairs(const int32_t* rounds, int n_pairs, int n_wg, int32_t* wg_begin, int32_t* seg_first,
                      int32_t* seg_count) {
  int n_used = 0;
  for (int p = 0; p < n_pairs; ++p) n_used += rounds[p] > 0;
  int w = 0, us = 0, k = 0;                                // share w is the next whose begin is not set yet
  for (int p = 0; p < n_pairs; ++p) {
    seg_first[p] = seg_count[p] = 0;
    if (rounds[p] == 0) continue;
    const int at = (int)((int64_t)k++ * n_wg / n_used);    // k-th pair with units: share k * n_wg / n_used
    while (w <= at) wg_begin[w++] = us;
    us += rounds[p] + kPairOverheadUnits;
    seg_first[p] = at;
    seg_count[p] = 1;
  }
  while (w <= n_wg) wg_begin[w++] = us;
}

// Where a list of whole pairs takes over from one of shares.  It saves the partials and their merge (a launch, or 1 to 2 us at the end
// of this one, merges_in_launch)
// and costs the time that the longest pair takes one CU beyond an even share of all rows.
// Tiled stores: the difference in us, whole pairs minus shares, as a sum over what both depend on; the factors were fitted to 1277
// pairs of timings of a kernel with four wavefronts and the merge launch (1 to 64 sequences of 100 to 8000 tokens, even and ragged, groups
// 1 to 16, 1 to 256 pairs); limits on the rows alone, which had been measured at group 4, were up to 1.7 x slower at others.  With the present
// kernel and what list_is_whole adds, over 396 timings (nine shapes of 1 to 64 sequences, groups 1 to 16, 40 to 1300 tokens, decode and step,
// plain and blending) the kind picked is the slower one by 0.5 % on average and by more than 10 % five times.  (Beyond 800 rows of excess
// nothing was fitted.)
// Row-major stores have no wide form, so rounds of four tiles count: one always pays; bf16 without gates two up to group 4, three up to
// group 2; beyond that only pairs that fill the CUs about evenly.  These limits are of the kernel before the matrix instructions; with the
// present one they pick the slower kind by 1.5 % on average of 792 timings as above, by more than 10 % 43 times: of fp32 beyond group 4 with 65 to
// 128 tokens, and of groups up to 2 with 200 to 400 (measured while those ran on the matrix cores too). Whole / shares, us: fp32, one
// sequence, 16 heads on 1, 40 tokens 8.3 / 10.3, 100 11.6 / 10.4, 130 14.9 / 10.3; 32 on 8, half compressed, 100 5.0 / 5.6, 130 5.9 / 5.6,
// 260 7.8 / 5.8; bf16, the same, 130 5.4 / 6.3, 200 6.6 / 6.3, 260 7.2 / 6.3; 16 on 1, 100 10.9 / 12.9, 130 14.3 / 13.1; fp32, 64 of 28 and
// 4 heads that blend, 400 32.2 / 34.0; 32 of 64 and 4, 130 16.1 / 15.1.
struct WholeCost {
  double fixed;          // merge launch saved, start of eight wavefronts
  double longest, even;  // per 1000 rows of the longest pair; of an even share
  double alike;          // per doubling of the pairs as long as the longest: they share the memory
  double wide;           // group beyond 8
  double filled;         // per pair and CU: shares cut the more pairs in two, the nearer these are in number
};
constexpr WholeCost kWholeCost[2][2] = {      // [some full head blends][planned by a fused step]
    {{-4.1, 3.9, -4.8, 0.4, 0.4, -1.3}, {-4.1, 3.9, -3.9, 0.4, 0.3, -2.1}},
    {{-2.9, 3.8, -3.9, 0.1, 0.4, -1.8}, {-3.3, 4.0, -3.2, 0.4, 0.8, -5.3}}};
constexpr double kInsideSaves = 1.2;
bool wants_whole_pairs(int kernel, int dtype, int group, bool gated, bool step, int n_wg, int n_kv_heads, int n_full, int window,
                       int batch, const int32_t* lengths, const uint8_t* active, bool merged_inside) {
  int64_t pairs = 0, longest = 0, all = 0;
  for (int b = 0; b < batch; ++b) {
    if (active && !active[b]) continue;
    pairs += n_kv_heads;
    const int64_t n = lengths[b], n_comp = std::min<int64_t>(n, window);
    longest = std::max(longest, n_full > 0 ? n : n_comp);
    all += n_full * n + (n_kv_heads - n_full) * n_comp;
  }
  if (pairs > n_wg) return false;
  const int64_t excess = longest - all / n_wg;
  if (kernel != RLKV_KERNEL_MFMA) {
    const bool light = group <= 4 && !gated;
    const int rounds = !light || dtype == RLKV_F32 ? 1 : group <= 2 ? 3 : 2;
    return longest <= rounds * kRound * kTile || excess <= (light ? 128 : 64);
  }
  if (longest == 0) return true;
  const WholeCost& c = kWholeCost[gated][step];
  const double diff = c.fixed + (c.longest * longest + c.even * all / n_wg) * 1e-3 + c.alike * std::log2(1.0 + (double)all / longest) +
                      (group > 8 ? c.wide : 0.0) + c.filled * pairs / n_wg;
  return excess <= 800 && diff + (merged_inside ? kInsideSaves : 0.0) <= 0.0;
}

// The kind of list a layer gets (true: whole pairs).  wants_whole_pairs was fitted with a merge launch behind the shares; where the
// tiled kernel merges them itself (merges_in_launch in rlkv_api.hip), they are better by kInsideSaves, and a list that goes out at one
// round per workgroup and fills at most half of the grid is one of shares beyond 352 rows, where heads blend beyond 256, which the eight
// wavefronts take in one go.  Whole / shares, us, decode and step: one sequence, 32 on 8 heads, half compressed, 230 tokens 4.1 / 4.9 and
// 5.2 / 5.8, 300 4.4 / 4.9 and 5.4 / 5.5, 350 4.4 / 4.9 and 5.2 / 5.8, 1000 6.8 / 5.3 and 7.6 / 6.1; 8 of 28 on 4, 230 4.3 / 5.4 and 5.5 / 6.2, 350
// 5.7 / 5.6 and 6.3 / 6.2, 400 6.0 / 5.5 and 7.2 / 6.1; with heads that blend, 230 6.6 / 7.5 and 7.7 / 8.4, 260 7.3 / 7.4 and 8.1 / 8.0, 350 7.9 / 7.6 and
// 8.8 / 8.6, 400 9.3 / 7.5 and 10.1 / 8.2.
bool list_is_whole(int kernel, int dtype, int group, bool gated, bool step, int n_wg, int n_kv_heads, int n_full, int window,
                   int batch, const int32_t* lengths, const uint8_t* active) {
  const bool tiled = kernel == RLKV_KERNEL_MFMA;
  if (tiled) {
    auto rounds = [&](int64_t n) { return (n + kWorklistSlack + kTile * kRound - 1) / (kTile * kRound); };
    int64_t longest = 0, all = 0;                            // rows of the longest pair; rounds of all
    for (int b = 0; b < batch; ++b) {
      if (active && !active[b]) continue;
      const int64_t ring = std::min(lengths[b], window);
      longest = std::max<int64_t>(longest, n_full > 0 ? lengths[b] : ring);
      all += n_full * rounds(lengths[b]) + (n_kv_heads - n_full) * rounds(ring);
    }
    if (longest > (gated ? 256 : 352) && rounds(longest) <= 16 && 2 * all <= n_wg) return false;
  }
  return wants_whole_pairs(kernel, dtype, group, gated, step, n_wg, n_kv_heads, n_full, window, batch, lengths, active,
                           tiled && group <= 8 && !gated);
}

}  // namespace rlkv

extern "C" int32_t rlkv_plan_shares(const int32_t* rounds, int32_t n_pairs, int32_t n_workgroups, int32_t* wg_begin,
                                    int32_t* seg_first, int32_t* seg_count) {
  if (!rounds || !wg_begin || !seg_first || !seg_count || n_pairs < 1 || n_workgroups < 1) return -1;
  for (int p = 0; p < n_pairs; ++p)
    if (rounds[p] < 0 || rounds[p] > (1 << 24)) return -1;
  return rlkv::plan_shares(rounds, n_pairs, n_workgroups, wg_begin, seg_first, seg_count);
}

extern "C" int32_t rlkv_plan_prefill_form(int32_t n_compute_units, int32_t n_q_heads, int32_t n_kv_heads,
                                          int32_t n_full_heads, int32_t batch, const int32_t* n_tokens,
                                          const int32_t* cached, int32_t min_share_tiles, int32_t allow_narrow,
                                          int32_t* narrow, int32_t* n_split) {
  if (!n_tokens || !cached || !narrow || !n_split) return -1;
  if (n_compute_units < 1 || n_kv_heads < 1 || n_q_heads < n_kv_heads || n_q_heads % n_kv_heads != 0) return -1;
  if (n_full_heads < 0 || n_full_heads > n_kv_heads || batch < 1 || min_share_tiles < 1) return -1;
  using namespace rlkv;
  const int G = n_q_heads / n_kv_heads, per_block = G < 256 ? 256 / G : 1;     // chunk positions per workgroup
  int64_t blocks = 0, n_active = 0;
  int max_tok = 0, min_tiles = INT32_MAX;      // min_tiles: cached tiles of the shortest sequence that has a chunk
  for (int b = 0; b < batch; ++b) {
    if (n_tokens[b] < 0 || cached[b] < 0) return -1;
    if (n_tokens[b] == 0) continue;
    blocks += (n_tokens[b] + per_block - 1) / per_block;
    ++n_active;
    if (n_tokens[b] > max_tok) max_tok = n_tokens[b];
    if (cached[b] / kTile < min_tiles) min_tiles = cached[b] / kTile;
  }
  *narrow = 0;
  *n_split = 1;
  const int64_t long_wgs = blocks * (n_full_heads ? n_full_heads : n_kv_heads);
  if (n_active == 0 || 2 * long_wgs > n_compute_units) return 0;
  // (Dividing when the long workgroups need more than one round was measured and lost: three sequences of
  // the Qwen shape, 342 workgroups, 4.53 -> 4.76 ms per 16384 tokens.)
  constexpr int kMaxSplit = 8;
  const int64_t rows = (int64_t)((max_tok + per_block - 1) / per_block) * n_active * n_full_heads;   // slots per share
  for (int zc = 2; zc <= kMaxSplit && n_full_heads > 0; ++zc) {
    if (long_wgs * zc > n_compute_units || rows * zc > kPrefillSplitSlots || min_tiles / zc < min_share_tiles) break;
    *n_split = zc;
  }
  if (*n_split == 1 && allow_narrow) *narrow = 1;
  return 0;
}

namespace rlkv {

// Whether a chunk of a layer with blending heads takes the form with one column group per wavefront (128 columns to a workgroup) or
// two (256).  A workgroup of 128 columns takes about 0.6 of the time of one of 256, by three chunks of one batch (8 sequences of 1000
// to 4000 tokens, 28 query and 4 KV heads, chunks 1, 2, 3 of 1024: 44 / 71, 65 / 104, 79 / 130 us), so the wide form is the better one
// unless it fills its last round of workgroups so much worse.  (Dividing a half-empty round, which only the narrow form can, is not
// weighed.)
bool plan_blend_narrow(int n_compute_units, int group, int n_full_heads, int batch, const int32_t* n_tokens) {
  int64_t rounds[2];
  for (int form = 0; form < 2; ++form) {
    const int per_block = (form ? 128 : 256) / group;
    int64_t blocks = 0;
    for (int b = 0; b < batch; ++b) blocks += (n_tokens[b] + per_block - 1) / per_block;
    rounds[form] = (blocks * n_full_heads + n_compute_units - 1) / n_compute_units;
  }
  return 3 * rounds[1] < 5 * rounds[0];
}

// Shares that every full-head workgroup of a chunk is divided into in the form with one column group per wavefront (128 columns
// to a workgroup).  As above: only where the shares still fit the CUs in one round.
int plan_narrow_split(int n_compute_units, int group, int n_full_heads, int batch, const int32_t* n_tokens,
                      const int32_t* cached, int min_share_tiles) {
  const int per_block = 128 / group;
  int64_t blocks = 0, n_active = 0;
  int max_tok = 0, min_tiles = INT32_MAX;
  for (int b = 0; b < batch; ++b) {
    if (n_tokens[b] == 0) continue;
    blocks += (n_tokens[b] + per_block - 1) / per_block;
    ++n_active;
    if (n_tokens[b] > max_tok) max_tok = n_tokens[b];
    if (cached[b] / kTile < min_tiles) min_tiles = cached[b] / kTile;
  }
  const int64_t rows = (int64_t)((max_tok + per_block - 1) / per_block) * n_active * n_full_heads;
  int n_split = 1;
  constexpr int kMaxSplit = 8;
  for (int z = 2; z <= kMaxSplit && rows > 0; ++z) {
    if (blocks * n_full_heads * z > n_compute_units || rows * z > kPrefillSplitSlots || min_tiles / z < min_share_tiles) break;
    n_split = z;
  }
  return n_split;
}

int64_t plan_prefill_items(int per_block, int n_seqs, const int32_t* tokens, int gx, const int32_t (&n_heads)[2], int dealt_rows,
                           PrefillItems* items, int32_t* first) {
  int64_t blocks = (int64_t)n_seqs * gx;
  int whole = n_seqs;                                // leading sequences with gx blocks
  items->ragged = 0;
  if (tokens) {
    whole = 0;
    while (whole < n_seqs && (tokens[whole] + per_block - 1) / per_block == gx) ++whole;
    if (whole < n_seqs) {
      items->ragged = 1;
      blocks = 0;
      for (int i = 0; i < n_seqs; ++i) {
        first[i] = (int32_t)blocks;
        blocks += (tokens[i] + per_block - 1) / per_block;
      }
      first[n_seqs] = (int32_t)blocks;
      std::fill(first + n_seqs + 1, first + kFirstEntries, INT32_MAX);
    }
  }
  items->gx = gx;
  items->n_seqs = n_seqs;
  items->inv_gx = quotient_inverse(gx);
  for (int c = 0; c < 2; ++c) {
    items->heads[c] = n_heads[c];
    items->inv_heads[c] = quotient_inverse(n_heads[c]);
    items->inv_seq[c] = quotient_inverse(n_heads[c] * gx);
  }
  items->dealt[0] = std::min(dealt_rows, whole * n_heads[0]) / 8 * 8;
  items->dealt[1] = whole * n_heads[1] / 8 * 8;
  items->rest = (int32_t)(blocks * n_heads[0] - (int64_t)items->dealt[0] * gx);
  return blocks * (n_heads[0] + n_heads[1]);
}

}  // namespace rlkv

extern "C" int32_t rlkv_plan_prefill_rows(int32_t n_full_heads, int32_t batch, const int32_t* n_tokens,
                                          const int32_t* cached, int32_t* dealt_rows, int32_t* heavy_rows) {
  if (!n_tokens || !cached || !dealt_rows || !heavy_rows || n_full_heads < 0 || batch < 1) return -1;
  // work of a full head's grid row: its queries times the keys each attends over on average, plus a constant
  // per query for what a workgroup costs beside its unmasked tiles; sequences in the order of the grid
  // (those with a chunk first, then by cached + chunk length, longest first; stable)
  std::vector<int32_t> order;
  for (int b = 0; b < batch; ++b) {
    if (n_tokens[b] < 0 || cached[b] < 0) return -1;
    if (n_tokens[b] > 0) order.push_back(b);
  }
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
    return (int64_t)cached[x] + n_tokens[x] > (int64_t)cached[y] + n_tokens[y];
  });
  const int heavy = (int)order.size() * n_full_heads;
  auto work = [&](int row) {
    const int32_t b = order[row / n_full_heads];
    return (double)n_tokens[b] * ((double)cached[b] + 0.5 * n_tokens[b] + 600.0);
  };
  int dealt = 0;
  while (dealt + 8 <= heavy && work(dealt + 7) >= 0.85 * work(dealt)) dealt += 8;
  *dealt_rows = dealt;
  *heavy_rows = heavy;
  return 0;
}

extern "C" int32_t rlkv_plan_prefill_block(int32_t linear_index, int32_t grid_x, int32_t grid_y, int32_t dealt_rows,
                                           int32_t heavy_rows, int32_t* block_x, int32_t* block_y) {
  if (!block_x || !block_y || grid_x < 1 || grid_y < 1 || linear_index < 0 ||
      (int64_t)linear_index >= (int64_t)grid_x * grid_y)
    return -1;
  // rows of grid_x blocks each, the heavy ones first
  const int heavy = heavy_rows < grid_y ? std::max(heavy_rows, 0) : grid_y;
  const int dealt = std::min(std::max(dealt_rows, 0), heavy) / 8 * 8;
  rlkv::PrefillItems items = {};
  items.gx = grid_x;
  items.dealt[0] = dealt;
  items.dealt[1] = (grid_y - heavy) / 8 * 8;
  items.rest = (heavy - dealt) * grid_x;
  items.inv_gx = rlkv::quotient_inverse(grid_x);
  int index = 0;
  if (!rlkv::prefill_item(linear_index, items, index)) index += heavy * grid_x;
  *block_x = index % grid_x;
  *block_y = index / grid_x;
  return 0;
}

extern "C" int32_t rlkv_plan_prefill_item(int32_t linear_index, int32_t per_block, int32_t n_full_heads, int32_t n_compressed_heads,
                                          int32_t n_seqs, const int32_t* n_tokens, int32_t dealt_rows, int32_t* item) {
  if (!n_tokens || !item || per_block < 1 || n_full_heads < 0 || n_compressed_heads < 0 || n_seqs < 1 || n_seqs > rlkv::kArgSeqs ||
      dealt_rows < 0 || linear_index < 0)
    return -1;
  int32_t longest = 0;
  for (int i = 0; i < n_seqs; ++i) {
    if (n_tokens[i] < 1) return -1;
    longest = std::max(longest, n_tokens[i]);
  }
  const int32_t n_heads[2] = {n_full_heads, n_compressed_heads};
  rlkv::PrefillItems items;
  int32_t first[rlkv::kFirstEntries];
  const int gx = (longest + per_block - 1) / per_block;
  if (linear_index >= rlkv::plan_prefill_items(per_block, n_seqs, n_tokens, gx, n_heads, dealt_rows, &items, first)) return 1;
  int index = 0, place = 0, head = 0, block = 0, blocks = gx;
  const bool full = rlkv::prefill_item(linear_index, items, index);
  if (items.ragged) {
    const int c = full ? 0 : 1;
    const int x = rlkv::quotient(index, items.heads[c], items.inv_heads[c]);
    while (first[place + 1] <= x) ++place;
    blocks = first[place + 1] - first[place];
    rlkv::ragged_place(index, items.heads[c], first[place], blocks, head, block);
  } else {
    rlkv::even_place(index, full, items, place, head, block);
  }
  item[0] = full;
  item[1] = place;
  item[2] = head;
  item[3] = blocks - 1 - block;
  return 0;
}

extern "C" int32_t rlkv_plan_whole_pairs(const int32_t* rounds, int32_t n_pairs, int32_t n_workgroups, int32_t* wg_begin,
                                         int32_t* seg_first, int32_t* seg_count) {
  if (!rounds || !wg_begin || !seg_first || !seg_count || n_pairs < 1 || n_workgroups < 1) return -1;
  int used = 0;
  for (int p = 0; p < n_pairs; ++p) {
    if (rounds[p] < 0 || rounds[p] > (1 << 24)) return -1;
    used += rounds[p] > 0;
  }
  if (used > n_workgroups) return -1;
  rlkv::plan_whole_pairs(rounds, n_pairs, n_workgroups, wg_begin, seg_first, seg_count);
  return used;
}

static bool list_arguments_valid(int32_t kernel, int32_t dtype, int32_t group, int32_t n_workgroups, int32_t n_kv_heads, int32_t n_full_heads,
                                 int32_t window, int32_t batch, const int32_t* lengths) {
  if (!lengths || (kernel != RLKV_KERNEL_VALU && kernel != RLKV_KERNEL_MFMA) || (dtype != RLKV_F32 && dtype != RLKV_BF16)) return false;
  if (group < 1 || group > rlkv::kMaxGroup || n_workgroups < 1 || n_kv_heads < 1 || n_full_heads < 0 || n_full_heads > n_kv_heads ||
      window < 1 || batch < 1)
    return false;
  for (int b = 0; b < batch; ++b)
    if (lengths[b] < 0) return false;
  return true;
}

extern "C" int32_t rlkv_plan_list_whole(int32_t kernel, int32_t dtype, int32_t group, int32_t gated, int32_t step, int32_t n_workgroups,
                                        int32_t n_kv_heads, int32_t n_full_heads, int32_t window, int32_t batch,
                                        const int32_t* lengths, const uint8_t* active) {
  if (!list_arguments_valid(kernel, dtype, group, n_workgroups, n_kv_heads, n_full_heads, window, batch, lengths)) return -1;
  return rlkv::wants_whole_pairs(kernel, dtype, group, gated != 0, step != 0, n_workgroups, n_kv_heads, n_full_heads, window, batch,
                                 lengths, active, false);
}

extern "C" int32_t rlkv_plan_list_kind(int32_t kernel, int32_t dtype, int32_t group, int32_t gated, int32_t step, int32_t n_workgroups,
                                       int32_t n_kv_heads, int32_t n_full_heads, int32_t window, int32_t batch,
                                       const int32_t* lengths, const uint8_t* active) {
  if (!list_arguments_valid(kernel, dtype, group, n_workgroups, n_kv_heads, n_full_heads, window, batch, lengths)) return -1;
  return rlkv::list_is_whole(kernel, dtype, group, gated != 0, step != 0, n_workgroups, n_kv_heads, n_full_heads, window, batch,
                             lengths, active);
}

extern "C" int32_t rlkv_plan_blend_form(int32_t n_compute_units, int32_t group, int32_t n_full_heads, int32_t batch,
                                        const int32_t* n_tokens, int32_t allow_narrow) {
  if (!n_tokens || n_compute_units < 1 || group < 1 || group > rlkv::kMaxGroup || n_full_heads < 0 || batch < 1) return -1;
  for (int b = 0; b < batch; ++b)
    if (n_tokens[b] < 0) return -1;
  return allow_narrow && rlkv::plan_blend_narrow(n_compute_units, group, n_full_heads, batch, n_tokens);
}

extern "C" int32_t rlkv_plan_narrow_split(int32_t n_compute_units, int32_t group, int32_t n_full_heads, int32_t batch,
                                          const int32_t* n_tokens, const int32_t* cached, int32_t min_share_tiles) {
  if (!n_tokens || !cached || n_compute_units < 1 || group < 1 || group > rlkv::kMaxGroup || n_full_heads < 0 || batch < 1 ||
      min_share_tiles < 1)
    return -1;
  for (int b = 0; b < batch; ++b)
    if (n_tokens[b] < 0 || cached[b] < 0) return -1;
  return rlkv::plan_narrow_split(n_compute_units, group, n_full_heads, batch, n_tokens, cached, min_share_tiles);
}
