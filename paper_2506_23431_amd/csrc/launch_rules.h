// Launch shapes that follow from sizes alone: host code without device types, so that it can be compiled and checked by
// itself.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

// ---------------------------------------------------------------------------
// Attention: work-groups per (request, head, query group) and waves per work-group.
// ---------------------------------------------------------------------------
struct AttnShape { int splits, waves; };

// units: (request, head, query group) triples; nblk: 32-key blocks, of a decode step those of the middle of its run; cap:
// splits the partials' buffer has room for; decode: a step (few rows per request), not a context pass; pair: keys and
// values are pairs of halves; streamed: what a step reads at full capacity passes the last-level cache.
// One work-group of 4 waves per unit; the same with 8 waves; or splits of 4 waves, about one work-group per compute unit
// and at least one key block per wave, and the merge kernel.  The estimate of each, in us: the key blocks of a wave one
// after the other, each at the slowest of three paces (measured at head sizes 32-128, 4-256 units, 4-104 blocks):
//   what a wave alone needs, 0.55 (1.1 where the caches do not hold the keys);
//   its share of what a compute unit draws, 105 (60) KB per us;
//   its share of what the device delivers, 13 (9) GB per ms, 8 % more with 8 waves asking.
// The merge kernel costs 3.4, and 8 waves end 0.1 + 0.005 head_dim later than 4.  So splits take over from 8 waves at 46
// blocks for 8 units of head size 64 from the caches, 31 from memory, 20 at head size 96 and 17 at 128 (us per layer and
// step, 8 waves / splits: head size 64 from the caches 48 blocks 25.3 / 25.4, 72 blocks 26.9 / 25.5; 16 units from memory
// 40 blocks 33.7 / 32.1; head size 128, 8 units 32 blocks 36.6 / 32.6, 16 units 64 blocks 56.5 / 44.0).  The choice is
// within 1.1 us of the best of the three at all 900 points, 0.04 on average; with one pace of 0.55 us per block for every
// head size it was up to 12.5 off, 1.06 on average.  Fewer blocks than waves: 4 waves (5 blocks 0.3-1.1 us better).  More units than
// compute units: 4 waves do as well or better (288 units x 384 keys, 12 steps 4.46 against 4.51 ms); beyond 96 blocks a
// unit's keys want more than one compute unit's share (128 units x 4096-6000 keys, 40 steps: 52.9 against 51.7 ms).
// Splits: a work-group per compute unit, every wave streaming several key blocks back to back (16 heads x 8k keys 16.2 us
// with 256 work-groups, 17.2 with 512 or 768, 18.7 with 320; 4 x 32 heads x 4k keys 256 are 4 us per launch faster than
// 768).  Context passes and pair layers: one work-group up to 32 blocks, then splits.
inline AttnShape attn_shape(int head_dim, int units, int nblk, int cap, bool decode, bool pair, bool streamed) {
  const int splits = std::max(1, std::min(std::min(std::max(1, 256 / units), std::max(1, nblk / 4)), cap));
  if (!decode || pair) return AttnShape{nblk <= 32 ? 1 : splits, 4};
  const double kb = 0.128 * head_dim;
  auto pace = [&](int waves, int groups) {
    const double device = (streamed ? 9e3 : 13e3) * (waves == 8 ? 1.08 : 1.0);
    return std::max({streamed ? 1.1 : 0.55, waves * kb / (streamed ? 60.0 : 105.0), groups * waves * kb / device});
  };
  AttnShape best{1, 4};
  double us = nblk / 4.0 * pace(4, units);
  if (nblk >= 8 && nblk <= 96 && units <= 256) {
    const double t = nblk / 8.0 * pace(8, units) + 0.1 + 0.005 * head_dim;
    if (t < us) { us = t; best = AttnShape{1, 8}; }
  }
  if (splits > 1 && 3.4 + nblk / (4.0 * splits) * pace(4, units * splits) < us) best = AttnShape{splits, 4};
  return best;
}

// ---------------------------------------------------------------------------
// Teacher-forced pass: consecutive requests that share launches, their rows padded to the longest of the group.
// ---------------------------------------------------------------------------
struct PassCost { double pass_us, row_us; };

// What a pass costs whatever its rows (9 launches per layer and a few more at 4 us, the weights once at 4.5 TB/s) and per
// row (multiplies at 0.6 PFLOP/s).  weights: elements of all matrices; parts: 2 with low parts, else 1.  Measured, per
// call and row: 2 layers of width 2048, 32000 words 227 us at 8 rows, +0.74 us per row (estimate 158 + 1.1); 6 of
// width 768, 2000 words 269 us, +0.37 (232 + 0.29); 4 of width 1024 230 us, +0.38 (190 + 0.39).
inline PassCost teacher_pass_cost(int n_layer, double weights, int parts) {
  return PassCost{4.0 * (9 * n_layer + 5) + 2.0 * weights / 4.5e6, 2.0 * parts * weights / 0.6e9};
}

// Sizes of the groups: the consecutive partition with the least estimated time.  fits(rows per request, requests) says
// what one launch sequence holds (not more requests where fewer did not fit).  One request of 500 rows before
// seven of 20 is a pass of its own in wide models (padded they would be 4000 rows where 640 carry a token) and shares
// in narrow ones, where a pass costs more than the padding.
template <typename Fits>
inline std::vector<int> teacher_groups(const std::vector<int> &rows, const PassCost &cost, Fits fits) {
  constexpr int MOST = 1024;            // requests of a group (bounds the search; such a pass has as many rows)
  const int n = (int)rows.size();
  std::vector<double> best(n + 1, 0.0);
  std::vector<int> size(n + 1, 0);
  for (int i = n - 1; i >= 0; --i) {    // best[i]: requests i .. n-1
    int longest = 0;
    best[i] = -1.0;
    for (int k = 1; i + k <= n && k <= MOST; ++k) {
      longest = std::max(longest, rows[i + k - 1]);
      if (k > 1 && !fits(longest, k)) break;
      const double t = cost.pass_us + cost.row_us * (double)k * longest + best[i + k];
      if (best[i] < 0 || t < best[i]) { best[i] = t; size[i] = k; }
    }
  }
  std::vector<int> groups;
  for (int i = 0; i < n; i += size[i]) groups.push_back(size[i]);
  return groups;
}
