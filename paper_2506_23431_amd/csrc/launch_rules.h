// Launch shapes that follow from sizes alone: host code without device types, so that it can be compiled and checked by
// itself.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
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
// head size it was up to 12.5 off, 1.06 on average.  Fewer blocks than waves: 4 waves (5 blocks 0.3-1.1 us better).  More
// units than compute units: 4 waves do as well or better (288 units x 384 keys, 12 steps 4.46 against 4.51 ms); beyond 96
// blocks a unit's keys want more than one compute unit's share (128 units x 4096-6000 keys, 40 steps: 52.9 against 51.7 ms).
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

// Two blocks per unit, each with half of the dims of the values, where one block per unit leaves half of the chip idle (us
// per launch, one block / two: 12 units of head size 64, 32-48 key blocks 6.6 / 6.1; 24 units, 22 blocks 6.0 / 5.4; 12 units, 16
// blocks 4.7 / 4.4, 1-5 blocks with 4 waves 4.2 / 4.0; 128 units, 64 blocks from memory 16.5 / 14.2).  Beyond 128 units the second
// blocks wait for the first.  In whole steps less of it is left: 2-128 units, 16-4000 keys, us gained per launch at head
// sizes 96 and 128 0.22 and 0.25 on average (-0.8 to 2.5), at 32 and 64 0.14 and 0.00 with 12 layers (-0.6 to 0.6) and -0.13 and
// -0.04 with 3, which is what runs of one side differ by.  attn_shape weighs 8 waves without halves against splits.
inline bool attn_halves(const AttnShape &shape, int units, bool decode, bool pair) {
  return shape.splits == 1 && units <= 128 && decode && !pair;
}

// ---------------------------------------------------------------------------
// Sizes that a projection kernel gets as leading arguments (four words beside five pointers fill the registers that a
// wave starts with), wide enough for every size that a context can have.
// ---------------------------------------------------------------------------
struct GemmWords {
  uint32_t lo;          // way from the activations to their low parts, in units of 64 values
  uint32_t k, share;    // k-tiles, and those of a wave (or of a block): 24 bits
  uint32_t n;           // column tiles | c2 follows c1 (bit 31) | row sums of 8 columns (bit 30); of a projection that prepares a
                        // norm: tiles | last row << 16
};
constexpr GemmWords gemm_words(int64_t lo_values, int K, int k_share, int n_tiles, bool c2, bool half_sums = false) {
  return GemmWords{(uint32_t)(lo_values / 64), (uint32_t)(K / 32), (uint32_t)k_share,
                   (uint32_t)n_tiles | (c2 ? 1u << 31 : 0u) | (half_sums ? 1u << 30 : 0u)};
}
constexpr GemmWords gemm_words_rows(int64_t lo_values, int K, int k_share, int n_tiles, int rows) {
  return GemmWords{(uint32_t)(lo_values / 64), (uint32_t)(K / 32), (uint32_t)k_share,
                   (uint32_t)n_tiles | (uint32_t)(rows > 0 ? rows - 1 : 0) << 16};
}
// (2^29 inner values, of which 128 rows are 275 GB.  That the compiler knows the range keeps what stands in front of the first
// requests short: without it the projections that finish a norm waited for the argument struct before they asked for the row
// sums, QKV of width 768 4.1 -> 4.2 us.)
constexpr int WORDS_K_TILES = 0xffffff;
constexpr int words_k_tiles(uint32_t k) { return (int)(k & WORDS_K_TILES); }
constexpr size_t words_granules(uint32_t lo) { return (size_t)lo * 8; }      // in 16-byte granules of 8 values
constexpr int words_tiles(uint32_t n) { return (int)(n & 0x3fffffffu); }
constexpr int words_half_sums(uint32_t n) { return (int)(n >> 30 & 1u); }
constexpr bool words_c2(uint32_t n) { return n >> 31; }
constexpr int words_tiles_rows(uint32_t n) { return (int)(n & 0xffffu); }
constexpr int words_last_row(uint32_t n) { return (int)(n >> 16); }

// ... and an attention kernel: heads (widths end at 8192, heads start at 32) and rows of a request (fewer than its cache
// slots, which end at 2^24) in one word.
constexpr uint32_t heads_rows(int H, int A) { return (uint32_t)(H - 1) | (uint32_t)A << 8; }
constexpr int word_heads(uint32_t w) { return (int)(w & 0xff) + 1; }
constexpr int word_rows(uint32_t w) { return (int)(w >> 8); }

// ---------------------------------------------------------------------------
// Steps of at most 16 rows: whether the second FFN projection prepares the next layer's first norm.
// ---------------------------------------------------------------------------
// It has to give up its cut along K over blocks for this, which leaves one block per 16 output columns, or per 8 in halves of
// tiles (k_gemm_half, which takes rows with low parts and inner values in pairs of k-tiles).  While a wave of 16 holds at most 8
// k-tiles (d_ff 4096) whole tiles cost less than the norm kernel (768 / 3072, whole steps: 174.6 against 184.1 us; 1024 / 4096
// 273 against 289; 512 / 1376 with rotary positions 186 against 204; encoder-decoder 1024 / 4096 22.5 against 22.9 ms per
// example), also where the 5 or 7 k-tiles of a wave take two batches of requests; halves gain no more there (us per step, whole /
// halves: width 512 181.3 / 182.3, 768 161.7 / 163.4, 1024 161.0 / 165.1).  Beyond width 1024 whole tiles leave too few blocks and
// halves are the better: us per step with the norm kernel / whole tiles / halves, 8 rows, weights in the last-level cache:
// width 1280, d_ff 3456 gated 208.8 / 193.9 / 193.7, 5120 210.8 / 196.2 / 194.5, 1536, 6144 146.4 / 139.3 / 135.6 (16 rows 161.5 /
// 156.2 / 155.3), 2048, 5504 gated 176.3 / 170.5 / 168.4; from memory, 12 layers: 1536, 6144 391.2 / 395.3 / 386.5, 2048, 5504
// 479.6 / 481.9 / 474.0.  At 2048, 8192 they gain from the cache (171.3 / 167.7 / 165.3) and lose from memory (1152.6 / 1195.7 /
// 1170.8): a block's activations, 32 bytes per inner value, outweigh the launch saved.
enum NormHandover { HANDOVER_NONE = 0, HANDOVER_WHOLE = 1, HANDOVER_HALVES = 2 };
inline NormHandover ffn2_handover(int d_model, int d_ff, bool low_parts, bool on_request) {
  if (d_model > 1024 && d_model <= 2048 && d_ff <= 6144 && d_ff % 64 == 0 && low_parts) return HANDOVER_HALVES;
  return (d_model <= 1024 && d_ff <= 4096) || on_request ? HANDOVER_WHOLE : HANDOVER_NONE;
}

// Room for the row sums (two values each) that projections of at most 128 rows leave: of every 16 columns and, at most 16 rows,
// behind 16 such rows of every 8.
constexpr size_t half_sums_at(int d_model) { return (size_t)16 * (d_model / 16); }
constexpr size_t norm_sums(int rows, int d_model) {
  const size_t whole = (size_t)(rows < 128 ? rows : 128) * (d_model / 16), halves = half_sums_at(d_model) + (size_t)16 * (d_model / 8);
  return whole > halves ? whole : halves;
}

// ---------------------------------------------------------------------------
// Steps that read more than the last-level cache holds: packed weights that are loaded without the non-temporal hint.
// ---------------------------------------------------------------------------
// What is loaded without the hint stays in that cache as long as it is little enough: the matrices, from layer 0 on, that start
// within the first 110 MB of the packed weights, unless they end beyond 210 MB.  With the hint on everything nothing survives a
// step, without it on more than the cache nothing does either.  Where the first line lies, ms per run of 20 steps with 0 / 60 / 90 / 110 / 130 / 170 / 220 MB kept: encoder-decoder of width
// 768, 12 layers 8.69 / 8.24 / 8.13 / 8.05 / 8.18 / 8.11 / 8.49, of 1024, 8 layers 6.62 / 6.39 / 6.31 / 6.23 / 6.27 / 6.58 / 6.96; 12
// layers of width 1024 7.34 / 7.05 / 6.98 / 6.93 / 7.09 / 6.99 / 6.90, 6 of 2048 5.47 / 5.29 / 5.27 / 5.26 / 5.38 / 5.42 / 5.43,
// 2 requests of 3000 keys, 6 of 1024 4.28 / 4.00 / 4.07 / 3.84 / 3.96 / 4.13 / 4.00; 24 of 2048 (4.4 GB a step) 0.3 %.
// Where the second one lies, us per step with the matrix that crosses the first kept / not (in brackets what is kept then):
// 2 layers of 3584 / 18944 gated [375 MB] 268.8 / 258.1, one of 2048 / 8192 before a head of 128000 words [625] 139.9 / 122.5, one of
// 8192 [402] 182.9 / 174.2, 4 of 3584 / 9728 gated [242] 347.6 / 351.3, with 4 requests of 2000 keys 495.9 / 485.5; 3 of 3328 / 8896
// gated [207] 256.9 / 260.2, with 8 requests of 4000 keys 542.0 / 547.4, 8 layers with 4 of 2000 879.1 / 864.3; one of 2048 before
// 26000 words [207] with 4 requests of 4000 keys 97.7 / 100.6, with 16 198.8 / 206.0; 3 of 3072 / 8192 gated [176] 223.5 / 225.8; 4 of
// 4096 / 11008 gated [134] 470.2 / 473.9.
constexpr size_t KEPT_START = 55000000, KEPT_END = 105000000;      // of 2 bytes
// first: values of packed weights before the matrix
constexpr bool weights_kept(size_t first, size_t values) { return first < KEPT_START && first + values <= KEPT_END; }

// ---------------------------------------------------------------------------
// fp32 projections: row tiles of 16 rows per block.
// ---------------------------------------------------------------------------
// A block of four row tiles reads a weight once for 64 rows, one of two for 32, at half of the registers; a row tile alone
// leaves its launch the most blocks.  Two or four want a block of two per compute unit and K beyond 256 (1024 x 256, 1000
// rows: one row tile 19.6 us, two 26.7, four 29.9).  Between them what counts is rounds of 256 blocks times the tiles of a block
// (6144 x 2048, 64 rows: 3 rounds of two 41 us, 2 of four 50; 4096 x 4096, 64 rows: 2 rounds of two 51, one of four 49).  Where
// these are equal, four are faster from K 2048 on (4096 x 11008, 512 rows 944 us against 1000; 3072 x 8192, 48 rows 82 against
// 89) and two below it (2048 x 512, 1000 rows 50 against 58); so are four in a single full round (4096 x 1024, 48 rows 15.0
// against 16.6), unless they pad more rows (2048 x 512, 80 rows 10.9 against 9.3).  At 460 sizes (K 64-11008, 40-1000 rows) two
// row tiles wherever they leave a block per compute unit are up to 1.14 times slower than four, and four up to 1.8 times slower
// than two; the rule is at most 1.08 times slower than the better of them (at K 64 0.8 us), with K up to 256 2 % faster on
// average.
inline int lin_row_tiles(int n_tiles, int K, int rows) {
  const long g2 = (rows + 31) / 32, g4 = (rows + 63) / 64;
  if (rows <= 32 || K <= 256 || n_tiles * g2 < 256) return 1;
  const long two = 2 * ((n_tiles * g2 + 255) / 256), four = 4 * ((n_tiles * g4 + 255) / 256);
  if (two != four) return two < four ? 2 : 4;
  if (four == 4) return g2 == 2 * g4 && K >= 512 ? 4 : 2;
  return K <= 2048 ? 2 : 4;
}

// ---------------------------------------------------------------------------
// fp32 attention: two blocks per (request, head, query group), each with all scores and half of the dims of the values.
// ---------------------------------------------------------------------------
// Where one block per unit leaves half of the chip idle: a block then draws three quarters of the bytes and multiplies three
// quarters (12 rows, 16 units of head size 64, 330 keys 11.7 -> 8.7 us).  us per step of 4 layers, one block / two: 320 keys of
// size 64, 8 units 130.3 / 122.3, 16 units 133.5 / 125.7, 200 keys, 64 units 128.5 / 127.4, 128 units 133.8 / 127.6, of size 80
// 160.3 / 152.7, 128 153.0 / 144.6.  With heads of 32 (109.6 / 114.2, 480 keys 109.1 / 112.1) or few keys (20 + generated 113.3 /
// 118.4) there is less to share than the second block costs, beyond 128 units the second blocks wait for the first.  The more
// keys, the more it gives, at every head size: 160 / 700 / 2000 keys, 8 units of size 64 0.91 / 0.89 / 0.85 of the time, 128 units
// 0.96 / 0.95 / 0.86, of size 128 0.94 / 0.88 / 0.83 and 0.96 / 0.90 / 0.82, of size 200 and 256 0.89-0.91 / 0.86; 160 units of size 64
// 1.07 / 1.12, 256 1.10.  Scalar loads (size 50) are even at 160 keys (0.99-1.02), 0.88-0.91 at 700.
inline bool attn_f32_halves(int head_dim, int units, int keys) { return head_dim > 32 && units <= 128 && keys >= 160; }

// ---------------------------------------------------------------------------
// fp32 steps of at most 32 rows: second FFN projection cut along K over 4 blocks.
// ---------------------------------------------------------------------------
// Uncut, a block per 16 columns draws its weights and rows through one compute unit; cut, whoever reads the rows next (QKV
// projection or head, a block per 16 columns and row tile, all of which normalise the rows) adds four slices.  Saved, in us: 0.9
// at d_ff 1024, where a wave of the uncut launch has two batches of requests, beyond 1.5 + 1.65 per 1024 (d_ff 2048 4.3,
// 8192 15).  Paid: 0.3, 1.0 and 2.4 for every round of 256 reading blocks at widths up to 256, 512 and 1024.  The next layer
// is one round or two; a head of 50000 words is 13 or 25 and costs more than any d_ff here saves at width 512 and beyond (one
// layer, us per step, uncut / cut: width 512, d_ff 2048, 12 rows, 500 words 50.3 / 47.9, 50000 words 89.7 / 98.7; width 1024,
// 32 rows, d_ff 1024, 50000 words 223 / 280; width 256, 8 rows, d_ff 4096, 50000 words 70.7 / 67.2).  At 1080 sizes (width 64-1024,
// d_ff 1024-8192, 1-32 rows, 500-50000 words) the choice costs 0.04 us more than the better one on average, 2.1 at most.
inline bool ffn2_in_slices(int d_model, int d_ff, int rows, int reader_tiles) {
  if (d_ff < 1024 || rows > 32 || d_model > 1024) return false;
  const double saved = d_ff > 1024 ? 1.5 + 1.65 * d_ff / 1024 : 0.9;
  const int rounds = (int)(((long)reader_tiles * (rows > 16 ? 2 : 1) + 255) / 256);
  return saved > rounds * (d_model <= 256 ? 0.3 : d_model <= 512 ? 1.0 : 2.4);
}

// ---------------------------------------------------------------------------
// Teacher-forced pass: consecutive requests that share launches, their rows padded to the longest of the group.
// ---------------------------------------------------------------------------
struct PassCost { double pass_us, row_us; };

// What a pass costs whatever its rows: 9 launches per layer and a few more at 4.3 us, the weights once at 2 TB/s (as the
// launches of few row tiles read them).  And per row: what norms, attention and epilogues take in a layer, its multiplies,
// the logits stored and read again for the loss.  layer, head: elements of a layer's and the vocabulary's matrices; parts:
// 2 with low parts, else 1.  Measured beyond 128 rows, per call (some 40 us of it outside the pass) and row: 6 layers of
// width 768, 2000 words 319 us, +0.46 per row (estimate 298 + 0.31), 50265 words 326, +0.71 (335 + 0.60); 4 of width 1024,
// 8000 words 306, +0.31 (235 + 0.32); 2 of 2048, 32000 words 322, +0.61 (265 + 0.59); 4 of 2048 / 5504 gated, 8000 words 459,
// +0.87 (395 + 0.86).
inline PassCost teacher_pass_cost(int n_layer, double layer, double head, int vocab, int parts) {
  return PassCost{4.3 * (9 * n_layer + 5) + (n_layer * layer + head) / 1e6,
                  n_layer * (0.025 + 1.75e-9 * parts * layer) + 6e-6 * vocab};
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

// ---------------------------------------------------------------------------
// Vocabulary projection of 33-128 rows with low parts: waves that share row tiles (k_gemm_t), or that cut K (k_gemm_s).
// ---------------------------------------------------------------------------
// k_gemm_s has two or four 16-word tiles per block and starts with every compute unit busy from 512 tiles on; each of its
// waves holds all row tiles of its K share, so weights arrive in as few, short batches as the registers leave room for.
// k_gemm_t has 8 or 16 tiles per block and streams the weights in order, but a block walks all of K: it wants
// a block per compute unit and more, and the more, the longer K is.  Both measured at 7 row counts, K 256-5120 and
// 1024-128000 words, weights from the caches and from memory; time of k_gemm_t over that of k_gemm_s, caches / memory.
// Beyond 80 rows (8 row tiles, one wave of k_gemm_s per SIMD): 0.50-0.92 from 1025 tiles on at every K, 0.93-1.5 at 1000
// tiles.  64 rows: K 768 1500 tiles 0.87 / 1.01, 2500 0.64 / 0.75; K 1536 1500 tiles 0.88 / 1.11, 2000 0.85 / 1.04, 2500
// 0.70 / 0.81; K 2048 1500 tiles 1.06 / 1.19, 2000 0.91 / 0.95; K 3072 2000 tiles 0.90 / 1.17.  Whole steps of one layer, its
// weights in the caches: width 768, 24000 words, 33 rows 54.1 -> 50.4 us, width 1024 58.7 -> 55.2.  By the sum of both
// times the line is within 3 % of the better kernel at 1065 of 1127 sizes, the others K 256 below it.
inline bool vocab_shares_row_tiles(int n_tiles, int KT, int rows) {
  return rows > 32 && (n_tiles >= 1500 + 12 * std::max(0, KT - 32) || (rows > 80 && n_tiles > 1024));
}

// ---------------------------------------------------------------------------
// Projections of more than 128 rows: kernel, tile and K slices of a launch.
// ---------------------------------------------------------------------------
// What a launch writes: K slices that the next norm kernel adds, activations or cache entries (of gate and up tiles one
// for two columns), winners (and logits).
enum RowOutput { ROWS_SLICES = 0, ROWS_STORED = 1, ROWS_VOCAB = 2, ROWS_GATED = 3 };

// cut: the waves of a block cut K (k_gemm_s), else they share row tiles (k_gemm_t); row and column tiles of a block (cut) or
// of a wave; K slices over blocks.
struct RowTiling { bool cut; int rt, nt, ks; };

// A tiling's time in us is the sum of c[.] times: 1; rounds of blocks as many as are resident at once (`resident` per
// compute unit, without / with low parts); those, and rounds of 256 blocks, times the k-tiles of a block; MB of weights and
// MB of activations that reach the L2 caches from beyond; million results written (slices, activations, vocabulary); GFLOP
// issued beyond 60, where launches run at the power limit and tiles differ in the operands they move per multiply.
// A column group's blocks sit on one XCD if the blocks of a row group are a multiple of 8, else on up to 8 of them, and
// every one fetches the weights; beyond 4 MB of weights per XCD they come again for every row group that is not in flight
// together.  Activations reach as many XCDs as a row group has column groups, at most 8.
// Coefficients with low parts: fit to 12000 launches inside context passes and decode steps (10 models of width 256-4096,
// 129-4096 rows, vocabularies of 1000-100000 words, every tiling in every place) and, with less weight, to 20000 by
// themselves whose weights cycle through 1.3 GB; without: to 25000 of the latter.  Chosen against the fastest of all
// candidates in the passes: 1.8 % slower on average, 1.0 % by total time.  An estimate fitted to 15 shapes, without terms
// for the fetches, was 12.6 and 23 % off: 2048 rows, K 3072, N 768 in slices took 40.7 us where 4 x 3 tiles take 30; 720
// rows, K 11008, N 4096 329 against 123; 256 rows, K 4096, 50304 words 582 against 187.
struct RowCost {
  bool cut;
  int rt, nt, resident[2];
  float c[2][10];
};
inline const RowCost *row_costs(int *n) {
  static const RowCost costs[] = {
      {true, 2, 2, {5, 4},
       {{2.03, 0, 0, 0.0351, 0.136, 0.0293, 0.493, 0.723, 0, 0},
        {2.81, 0, 0, 0.0512, 0.0527, 0.0493, 0.36, 1.26, 0.537, 0.11}}},
      {true, 2, 4, {1, 1},
       {{1.97, 0.318, 0.0558, 0, 0.0758, 0.0335, 0.999, 1.36, 0, 0},
        {2.67, 0.258, 0.0732, 0, 0.0688, 0.0658, 1.02, 2.08, 0.876, 0}}},
      {true, 2, 6, {2, 2},
       {{1.97, 0.807, 0.00982, 0.0612, 0.121, 0.0584, 0.243, 1.56, 0, 0},
        {3.41, 0.297, 0.00987, 0.0787, 0.0859, 0.0829, 0.252, 1.6, 0.609, 0}}},
      {false, 4, 1, {4, 3},
       {{2.19, 0, 0.182, 0.106, 0.0682, 0, 0.836, 1.31, 0, 0},
        {3.12, 0, 0.145, 0.147, 0.0388, 0.0161, 1.05, 1.49, 0.674, 0.13}}},
      {false, 4, 2, {2, 2},
       {{2.34, 0.573, 0.249, 0.119, 0.0837, 0.012, 0.663, 1.11, 0, 0},
        {2.91, 0.759, 0.182, 0.194, 0.0533, 0.033, 0.77, 1.44, 0.738, 0.109}}},
      {false, 4, 3, {2, 1},
       {{1.81, 2.23, 0.203, 0.218, 0.0892, 0.0452, 0.459, 1.16, 0, 0},
        {1.79, 3.06, 0.445, 0, 0.0484, 0.0551, 0.45, 1.38, 0.682, 0.0889}}},
      {false, 4, 4, {1, 1},
       {{4.22, 0.797, 0.498, 0, 0.0779, 0.0553, 0.374, 1.25, 0, 0},
        {2.68, 2.6, 0.572, 0, 0.0431, 0.0422, 0.609, 1.53, 1.1, 0.0739}}},
      {false, 8, 2, {1, 1},
       {{3.78, 1.45, 0.424, 0, 0.0637, 0.024, 0.437, 1.38, 0, 0},
        {2.15, 4.36, 0.577, 0, 0.0232, 0.0236, 0.564, 1.54, 0.725, 0.0795}}},
      {false, 8, 3, {1, 1},
       {{1.95, 5.22, 0.51, 0, 0.052, 0.0412, 0.285, 1.54, 0, 0},
        {0.954, 7.65, 0.771, 0, 0.0189, 0.0353, 0.384, 1.63, 0.709, 0.0803}}},
      {false, 8, 4, {1, 1},
       {{1.3, 7.83, 0.598, 0, 0.0619, 0.0436, 0.336, 1.66, 0, 0},
        {2.64, 7.52, 1.02, 0, 0.0117, 0.0368, 0.448, 1.74, 0.863, 0.0729}}}};
  *n = (int)(sizeof(costs) / sizeof(costs[0]));
  return costs;
}

inline double row_tiling_us(const RowCost &t, int n_tiles, int KT, int rows, int ks, bool split, RowOutput out) {
  const int wide = t.cut ? t.nt : 8 * t.nt, gx = (n_tiles + wide - 1) / wide, gz = (rows + 16 * t.rt - 1) / (16 * t.rt);
  const int group = gx * ks, kt = (KT + ks - 1) / ks, window = 256 * t.resident[split];
  const double blocks = (double)group * gz, w_mb = n_tiles * 16.0 * KT * 64e-6;
  const int xcds = group % 8 == 0 ? 1 : group % 4 == 0 ? 2 : group % 2 == 0 ? 4 : 8;
  const double together = std::max(1.0, (double)window / group);      // row groups in flight
  const double again = std::max(1.0, gz / together) * std::min((double)xcds, together);
  const double fetches = w_mb * xcds / 8 <= 4.0 ? std::min(xcds, gz) : std::min((double)gz, again);
  const double act_mb = (double)rows * KT * 64e-6 * (split ? 2 : 1) * std::min(8, gx);
  const double rounds = std::ceil(blocks / window), written = rows * (n_tiles * 16e-6) * (out == ROWS_GATED ? 0.5 : 1.0);
  const double power = std::max(0.0, rows * (n_tiles * 16.0) * KT * (split ? 128e-9 : 64e-9) - 60);
  const float *c = t.c[split];
  return c[0] + rounds * (c[1] + c[2] * kt) + std::ceil(blocks / 256) * kt * c[3] + c[4] * w_mb * fetches + c[5] * act_mb +
         c[out == ROWS_GATED ? 7 : 6 + out] * written * (out == ROWS_SLICES ? ks : 1) + c[9] * power;
}

inline RowTiling row_tiling(int n_tiles, int KT, int rows, int max_slices, bool split, RowOutput out) {
  int n;
  const RowCost *costs = row_costs(&n);
  RowTiling best{false, 8, 4, 1};
  double least = 1e30;
  for (int i = 0; i < n; ++i)
    for (int ks = 1; ks <= (out == ROWS_SLICES ? max_slices : 1); ks *= 2) {
      if (ks > 1 && KT / ks < 8) break;
      const double us = row_tiling_us(costs[i], n_tiles, KT, rows, ks, split, out) +
                        0.6 * (ks - 1) * rows * (double)n_tiles * 1.3e-5;      // what the next norm kernel pays for a slice
      if (us < least) { least = us; best = RowTiling{costs[i].cut, costs[i].rt, costs[i].nt, ks}; }
    }
  return best;
}
