// Launch shapes that follow from sizes alone: host code without device types, so that it can be compiled and checked by
// itself.
#pragma once
#include <stdint.h>

#include <algorithm>

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
