"""The rules by which launches are shaped (csrc/launch_rules.h), compiled by the host compiler alone: against times measured
for every shape a rule chooses from, and against exhaustive search where the rule is an optimum of its own estimate."""

import ctypes as C
import itertools
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_23431_amd", "csrc")

SOURCE = r"""
#include "launch_rules.h"
extern "C" {
void attn(int hd, int units, int nblk, int cap, int decode, int pair, int streamed, int *out) {
  const AttnShape s = attn_shape(hd, units, nblk, cap, decode, pair, streamed);
  out[0] = s.splits; out[1] = s.waves;
}
int groups(const int *rows, int n, double pass_us, double row_us, int row_cap, int most, int *out) {
  const std::vector<int> g = teacher_groups(std::vector<int>(rows, rows + n), PassCost{pass_us, row_us},
                                            [&](int a, int k) { return a * k <= row_cap && k <= most; });
  for (size_t i = 0; i < g.size(); ++i) out[i] = g[i];
  return (int)g.size();
}
void pass_cost(int n_layer, double layer, double head, int vocab, int parts, double *out) {
  const PassCost c = teacher_pass_cost(n_layer, layer, head, vocab, parts);
  out[0] = c.pass_us; out[1] = c.row_us;
}
void tiling(int n_tiles, int kt, int rows, int max_slices, int split, int kind, int *out) {
  const RowTiling t = row_tiling(n_tiles, kt, rows, max_slices, split, (RowOutput)kind);
  out[0] = t.cut; out[1] = t.rt; out[2] = t.nt; out[3] = t.ks;
}
int vocab(int n_tiles, int kt, int rows) { return vocab_shares_row_tiles(n_tiles, kt, rows); }
int lin(int n_tiles, int K, int rows) { return lin_row_tiles(n_tiles, K, rows); }
int64_t sums(int rows, int d) { return (int64_t)norm_sums(rows, d); }
int handover(int d, int ff, int low, int request) { return ffn2_handover(d, ff, low, request); }
int f32_halves(int hd, int units, int keys) { return attn_f32_halves(hd, units, keys); }
int kept(int64_t first, int64_t values) { return weights_kept(first, values); }
int slices(int d, int ff, int rows, int tiles) { return ffn2_in_slices(d, ff, rows, tiles); }
void words(int64_t lo, int K, int share, int n_tiles, int c2, int64_t *out) {
  const GemmWords w = gemm_words(lo, K, share, n_tiles, c2 & 1, c2 & 2);
  out[0] = words_granules(w.lo); out[1] = words_k_tiles(w.k); out[2] = words_k_tiles(w.share); out[3] = words_tiles(w.n); out[4] = words_c2(w.n); out[5] = words_half_sums(w.n);
}
int attn_word(int H, int A) {
  const uint32_t w = heads_rows(H, A);
  return word_heads(w) == H && word_rows(w) == A;
}
void words_rows(int64_t lo, int K, int share, int n_tiles, int rows, int64_t *out) {
  const GemmWords w = gemm_words_rows(lo, K, share, n_tiles, rows);
  out[0] = words_granules(w.lo); out[1] = words_k_tiles(w.k); out[2] = words_k_tiles(w.share); out[3] = words_tiles_rows(w.n); out[4] = 0;
  out[5] = words_last_row(w.n);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                           str(d / "rules.cpp"), "-o", str(d / "rules.so")])
    return C.CDLL(str(d / "rules.so"))


# head size, units, key blocks, keys from memory (else from the caches); us per layer and step with one work-group of 4
# waves per unit, of 8 waves, with splits and merge (3 layers, 4 rows per request)
ATTENTION = [
    (32, 8, 16, False, 22.8, 22.4, 24.9), (32, 8, 64, False, 27.4, 25.1, 24.9), (32, 64, 40, True, 32.5, 30.0, 31.2),
    (64, 4, 5, False, 21.6, 22.0, 21.7), (64, 8, 32, False, 25.4, 24.2, 25.2), (64, 8, 72, False, 29.8, 26.9, 25.5),
    (64, 16, 28, True, 33.6, 32.2, 32.1), (64, 16, 40, True, 35.9, 33.7, 32.1), (64, 64, 32, True, 35.1, 33.6, 34.2),
    (64, 64, 72, True, 43.4, 39.7, 37.6), (64, 128, 96, True, 54.9, 50.5, 51.2), (64, 256, 48, True, 49.8, 49.9, 49.8),
    (96, 8, 16, True, 30.8, 29.8, 31.1), (96, 16, 32, True, 34.6, 33.7, 31.7), (96, 64, 56, True, 45.9, 45.1, 42.1),
    (128, 4, 12, True, 27.6, 27.2, 28.6), (128, 8, 32, True, 37.0, 36.6, 32.6), (128, 16, 64, True, 56.7, 56.5, 44.0),
    (128, 32, 24, True, 37.5, 37.0, 35.4), (128, 64, 40, True, 45.9, 45.8, 43.2), (128, 128, 32, True, 55.8, 55.7, 57.2),
    (128, 128, 96, True, 77.2, 77.9, 76.4), (128, 256, 20, True, 66.9, 66.3, 66.5),
]


@pytest.mark.parametrize("hd,units,nblk,streamed,four,eight,split", ATTENTION)
def test_attention_shape_is_near_the_fastest_measured(rules, hd, units, nblk, streamed, four, eight, split):
    out = (C.c_int * 2)()
    rules.attn(hd, units, nblk, 4096 // units, 1, 0, int(streamed), out)
    splits, waves = out
    assert splits in (1, max(1, min(256 // units, nblk // 4))) and waves in (4, 8)
    us = split if splits > 1 else eight if waves == 8 else four
    assert us <= 1.03 * min(four, eight, split)


def test_attention_shape_at_its_limits(rules):
    out = (C.c_int * 2)()
    for hd, units, nblk, cap, streamed in itertools.product((32, 64, 96, 128), (1, 7, 64, 256, 257, 5000), (1, 4, 7, 8, 32, 33, 96, 97, 400),
                                                            (1, 3, 1000), (0, 1)):
        for decode, pair in ((1, 0), (0, 0), (1, 1)):
            rules.attn(hd, units, nblk, cap, decode, pair, streamed, out)
            assert 1 <= out[0] <= min(cap, max(1, nblk // 4))            # partials fit, every wave has a block
            if pair or not decode or nblk < 8 or nblk > 96 or units > 256:
                assert out[1] == 4
            if (pair or not decode) and nblk <= 32:
                assert out[0] == 1


def _groups(rules, rows, pass_us, row_us, row_cap=4096, most=1000):
    out = (C.c_int * len(rows))()
    n = rules.groups((C.c_int * len(rows))(*rows), len(rows), C.c_double(pass_us), C.c_double(row_us), row_cap, most, out)
    return list(out[:n])


def _cost(rows, groups, pass_us, row_us):
    total, at = 0.0, 0
    for k in groups:
        total += pass_us + row_us * k * max(rows[at:at + k])
        at += k
    assert at == len(rows)
    return total


def test_targets_share_a_pass_only_where_padding_costs_less(rules):
    wide = (265.0, 0.59)             # 2 layers of width 2048, 32000 words
    assert _groups(rules, [500] + [20] * 7, *wide) == [1, 7]
    assert _groups(rules, [20] * 7 + [500], *wide) == [7, 1]
    assert _groups(rules, [200, 190, 180], *wide) == [3]
    narrow = (232.0, 0.02)
    assert _groups(rules, [500] + [20] * 7, *narrow) == [8]
    cost = (C.c_double * 2)()
    rules.pass_cost(2, C.c_double(12 * 2048 ** 2), C.c_double(32000 * 2048), 32000, 2, cost)
    assert abs(cost[0] - wide[0]) < 1 and abs(cost[1] - wide[1]) < 0.01
    # 2 layers of width 2048, 8000 words, targets of 40 to 320 rows: one pass 1440 us, padded to 2560 rows; three passes 1640
    rules.pass_cost(2, C.c_double(12 * 2048 ** 2), C.c_double(8000 * 2048), 8000, 2, cost)
    assert len(_groups(rules, list(range(40, 321, 40)), cost[0], cost[1])) <= 2


def test_target_groups_are_the_cheapest_partition(rules):
    rng = np.random.default_rng(5)
    for _ in range(60):
        n = int(rng.integers(1, 9))
        rows = [int(r) for r in np.exp(rng.uniform(0, np.log(900), n))]
        pass_us, row_us, row_cap, most = float(rng.uniform(20, 400)), float(rng.uniform(0.05, 3)), 2048, int(rng.integers(2, 9))
        got = _groups(rules, rows, pass_us, row_us, row_cap, most)
        best = 1e30
        for cuts in itertools.product((0, 1), repeat=n - 1):
            sizes, run = [], 1
            for c in cuts:
                if c:
                    sizes.append(run)
                    run = 1
                else:
                    run += 1
            sizes.append(run)
            at, fits = 0, True
            for k in sizes:
                fits = fits and (k == 1 or (k <= most and k * max(rows[at:at + k]) <= row_cap))
                at += k
            if fits:
                best = min(best, _cost(rows, sizes, pass_us, row_us))
        at = 0
        for k in got:
            assert k == 1 or (k <= most and k * max(rows[at:at + k]) <= row_cap)
            at += k
        assert abs(_cost(rows, got, pass_us, row_us) - best) < 1e-6 * best


SLICES, STORED, VOCAB, GATED = 0, 1, 2, 3
# column tiles, k-tiles, rows, low parts, output; the candidates within 10 % of the fastest: (waves cut K, row tiles, column
# tiles, K slices): us
TILINGS = [
    (48, 96, 2048, True, SLICES, {(False, 4, 3, 4): 21.3}),
    (48, 96, 720, True, SLICES, {(False, 4, 2, 4): 14.1}),
    (256, 344, 720, True, SLICES, {(False, 8, 2, 2): 121.4, (False, 4, 2, 4): 121.9, (False, 8, 4, 4): 123.2,
                                   (False, 4, 2, 2): 128.7, (False, 4, 4, 2): 130.1, (False, 8, 2, 4): 132.2,
                                   (False, 4, 4, 4): 133.0}),
    (256, 344, 1280, True, SLICES, {(False, 8, 3, 2): 177.6}),
    (192, 24, 192, True, STORED, {(True, 2, 2, 1): 7.7, (True, 2, 4, 1): 7.8, (True, 2, 6, 1): 8.1}),
    (192, 24, 720, True, STORED, {(True, 2, 6, 1): 15.7, (True, 2, 2, 1): 16.0, (True, 2, 4, 1): 16.2,
                                  (False, 4, 1, 1): 16.6, (False, 4, 2, 1): 17.1}),
    (144, 24, 2048, True, STORED, {(False, 4, 3, 1): 23.6}),
    (1024, 128, 400, True, STORED, {(False, 4, 2, 1): 108.2, (False, 8, 2, 1): 109.8, (False, 4, 4, 1): 112.0}),
    (512, 64, 4096, True, STORED, {(False, 8, 4, 1): 224.2, (False, 4, 2, 1): 227.0, (False, 4, 4, 1): 236.7,
                                   (False, 8, 2, 1): 236.9}),
    (512, 64, 720, False, STORED, {(False, 4, 2, 1): 43.6, (False, 4, 1, 1): 44.4, (False, 8, 2, 1): 46.3}),
    (3144, 24, 192, True, VOCAB, {(False, 4, 1, 1): 45.2, (False, 4, 2, 1): 47.5, (False, 4, 3, 1): 49.4, (False, 8, 4, 1): 49.4}),
    (3144, 128, 256, True, VOCAB, {(False, 8, 4, 1): 186.8}),
    (3144, 24, 400, True, VOCAB, {(False, 4, 1, 1): 108.3, (False, 4, 2, 1): 109.5, (False, 8, 4, 1): 110.7, (False, 8, 2, 1): 116.3}),
    # inside context passes and decode steps
    (48, 24, 256, True, SLICES, {(True, 2, 2, 2): 4.8, (True, 2, 2, 1): 5.1, (True, 2, 4, 2): 5.1}),
    (48, 96, 2048, True, SLICES, {(False, 4, 3, 4): 25.5, (False, 4, 2, 2): 25.9, (False, 8, 2, 4): 26.9, (False, 4, 4, 4): 27.1}),
    (96, 192, 1280, True, SLICES, {(False, 4, 4, 4): 44.9, (False, 8, 2, 4): 46.2}),
    (128, 256, 400, True, SLICES, {(False, 4, 1, 4): 36.6, (False, 4, 2, 4): 39.1}),
    (256, 344, 2048, True, SLICES, {(False, 8, 4, 2): 249.4, (False, 4, 4, 1): 261.9}),
    (344, 32, 2048, True, GATED, {(False, 8, 3, 1): 46.0}),
    (512, 64, 900, True, STORED, {(False, 4, 2, 1): 58.7, (False, 4, 4, 1): 61.7, (False, 8, 2, 1): 62.0}),
    (384, 64, 4096, True, STORED, {(False, 8, 3, 1): 166.8, (False, 4, 2, 1): 168.4, (False, 4, 4, 1): 176.4, (False, 8, 2, 1): 178.8}),
    (3141, 24, 192, True, VOCAB, {(False, 4, 1, 1): 40.9, (False, 8, 4, 1): 44.5}),
    (1500, 32, 384, True, VOCAB, {(False, 8, 3, 1): 42.6}), (3141, 128, 256, True, VOCAB, {(False, 8, 4, 1): 162.1}),
]


@pytest.mark.parametrize("n_tiles,kt,rows,split,kind,near", TILINGS)
def test_row_tiling_is_near_the_fastest_measured(rules, n_tiles, kt, rows, split, kind, near):
    out = (C.c_int * 4)()
    rules.tiling(n_tiles, kt, rows, 4, int(split), kind, out)
    assert (bool(out[0]), *out[1:]) in near


def test_row_tiling_at_its_limits(rules):
    out = (C.c_int * 4)()
    known = {(1, 2, 2), (1, 2, 4), (1, 2, 6), (0, 4, 1), (0, 4, 2), (0, 4, 3), (0, 4, 4), (0, 8, 2), (0, 8, 3), (0, 8, 4)}
    for n_tiles, kt, rows, slices, split, kind in itertools.product((1, 6, 161, 8000), (1, 7, 8, 15, 16, 512), (129, 4096, 100000), (1, 2, 4),
                                                                    (0, 1), (0, 1, 2, 3)):
        rules.tiling(n_tiles, kt, rows, slices, split, kind, out)
        assert tuple(out[:3]) in known
        assert out[3] in ((1, 2, 4) if kind == SLICES else (1,)) and out[3] <= slices and (out[3] == 1 or kt // out[3] >= 8)


# column tiles, K, rows; us with waves that cut K and with waves that share row tiles, weights from the caches, then both from
# memory
VOCABULARY = [
    (1500, 768, 33, 13.4, 11.8, 15.1, 15.5), (1500, 768, 65, 15.3, 14.0, 17.0, 17.9), (1624, 768, 80, 16.8, 14.2, 18.1, 18.1),
    (2500, 768, 33, 25.2, 16.5, 27.2, 20.1), (1624, 1024, 65, 20.0, 17.8, 21.4, 20.7), (2000, 1536, 64, 24.4, 20.8, 27.0, 28.1),
    (1748, 1536, 33, 22.6, 19.7, 24.8, 26.7), (2500, 1536, 64, 37.8, 26.4, 42.8, 34.6), (2500, 2048, 80, 46.5, 38.1, 53.0, 46.8),
    (1000, 2048, 64, 20.6, 24.0, 20.0, 31.0), (2000, 2048, 64, 34.6, 31.5, 37.5, 35.8), (1500, 2048, 80, 26.7, 30.7, 30.2, 37.3),
    (3144, 768, 65, 31.5, 22.2, 34.5, 27.7), (1028, 768, 96, 24.0, 16.0, 25.8, 19.2), (1028, 5120, 128, 91.3, 70.7, 98.1, 90.4),
    (1000, 2048, 96, 26.2, 32.0, 28.3, 38.3), (1000, 768, 128, 14.7, 15.8, 16.2, 19.3),
    (3144, 1024, 128, 61.5, 35.2, 65.8, 36.6), (1500, 4096, 80, 40.7, 52.0, 47.0, 70.3),
]


@pytest.mark.parametrize("n_tiles,k,rows,cut,share,cut_cold,share_cold", VOCABULARY)
def test_vocabulary_kernel_is_the_faster_measured(rules, n_tiles, k, rows, cut, share, cut_cold, share_cold):
    cut, share = cut + cut_cold, share + share_cold
    assert (share if rules.vocab(n_tiles, k // 32, rows) else cut) <= 1.03 * min(cut, share)


def test_few_rows_keep_waves_that_cut_k(rules):
    assert not any(rules.vocab(n, kt, rows) for n, kt, rows in itertools.product((1, 1024, 8000, 20000), (1, 24, 128), (1, 16, 32)))


def test_words_of_a_projection_hold_every_size(rules):
    """What a projection kernel unpacks is what the launch packed, up to sizes that no memory holds: 2^29 inner values, a
    vocabulary of 2^31 words, low parts 2^38 values away."""
    out = (C.c_int64 * 6)()
    for lo, k, share, tiles, c2 in itertools.product((0, 64, 512, 1 << 33, (1 << 38) - 64), (32, 1 << 21, (1 << 29) - 32),
                                                     (1, 65535, 65536, (1 << 24) - 1), (1, (1 << 24) + 1, (1 << 28) - 1), (0, 1)):
        rules.words(C.c_int64(lo), k, share, tiles, c2, out)
        assert list(out) == [lo // 8, k // 32, share, tiles, c2, 0]
    for tiles, rows in itertools.product((1, 512, 65535), (0, 1, 2, 16, 128)):
        rules.words_rows(C.c_int64(64), 64, 2, tiles, rows, out)
        assert list(out) == [8, 2, 2, tiles, 0, max(rows - 1, 0)]


def test_word_of_an_attention_launch_holds_every_size(rules):
    for H, A in itertools.product((1, 2, 255, 256), (1, 65535, 65536, (1 << 24) - 1)):
        assert rules.attn_word(H, A)


# fp32 projections: N, K, rows; us with one, two and four row tiles of 16 rows per block
LINEAR = [
    (256, 256, 1000, 6.9, 9.0, 9.3), (1024, 256, 1000, 19.6, 26.7, 29.9), (512, 128, 512, 7.4, 11.5, 10.0),
    (512, 512, 128, 4.7, 6.0, 9.5), (512, 512, 512, 11.0, 10.3, 9.4), (1536, 512, 96, 9.1, 9.5, 11.5),
    (2048, 512, 80, 9.2, 9.3, 10.9), (2048, 512, 128, 13.3, 10.3, 11.1), (2048, 512, 1000, 60.8, 49.9, 58.2),
    (512, 2048, 128, 10.8, 14.8, 25.8), (512, 2048, 256, 18.2, 15.0, 25.8), (512, 2048, 1000, 63.2, 49.6, 49.6),
    (3072, 768, 48, 15.7, 16.2, 14.9), (4096, 1024, 48, 16.9, 16.6, 15.0), (1024, 4096, 64, 18.0, 25.1, 46.3),
    (1024, 4096, 128, 32.2, 25.6, 45.5), (6144, 2048, 64, 56.9, 41.4, 49.6), (2048, 2048, 96, 26.0, 26.6, 26.1),
    (2048, 5504, 96, 67.7, 67.4, 63.3), (2048, 5504, 1000, 684.0, 507.1, 486.1), (3072, 8192, 48, 91.8, 89.1, 82.3),
    (3072, 3072, 128, 71.9, 57.4, 73.0), (4096, 11008, 40, 131.9, 129.2, 112.9), (4096, 11008, 96, 252.0, 197.4, 219.1),
    (4096, 11008, 512, 1276.1, 999.8, 943.7), (12288, 4096, 64, 209.5, 143.9, 139.4), (11008, 4096, 128, 363.8, 249.4, 263.0),
]


def test_fp32_row_tiles_against_measured_times(rules):
    """The chosen number of row tiles is within a tenth of the fastest at every measured size (the two rules before it, two row
    tiles or four wherever they leave enough blocks, were up to 1.15 and 1.8 times the other's time here)."""
    for N, K, rows, *us in LINEAR:
        t = dict(zip((1, 2, 4), us))
        assert t[rules.lin((N + 15) // 16, K, rows)] <= 1.10 * min(t.values()), (N, K, rows)


def test_fp32_row_tiles_at_the_limits(rules):
    for n_tiles, K, rows in itertools.product((1, 2, 255, 256, 16000, 1 << 26), (1, 256, 257, 512, 2048, 2049, 1 << 20),
                                              (1, 32, 33, 64, 65, 8192, 2100000)):
        t = rules.lin(n_tiles, K, rows)
        assert t in (1, 2, 4) and (t == 1 or (rows > 32 and n_tiles * -(-rows // 32) >= 256))


# fp32 steps: width, d_ff, rows, words of the head that reads the rows next (0: the next layer's QKV projection); us per step
# with the second FFN projection in slices minus us without
FFN2 = [
    (64, 1024, 16, 500, 0.0), (64, 1024, 32, 50000, 6.1), (64, 2048, 8, 500, -3.5), (64, 2048, 17, 50000, 2.0),
    (64, 4096, 16, 50000, -5.0), (64, 8192, 32, 0, -17.3), (128, 1536, 16, 0, -3.7), (128, 1536, 32, 50000, 2.5),
    (256, 1024, 17, 50000, 8.2), (256, 2048, 32, 20000, -1.1), (256, 2048, 32, 50000, 5.6), (256, 4096, 8, 50000, -2.4),
    (512, 1024, 1, 50000, 12.1), (512, 1024, 8, 0, 0.0), (512, 2048, 16, 8000, -3.1), (512, 2048, 16, 0, -3.7),
    (512, 2048, 8, 50000, 8.0), (512, 4096, 32, 8000, -5.8), (512, 8192, 17, 50000, 5.4), (512, 8192, 16, 20000, -13.0),
    (768, 1024, 16, 0, 0.8), (768, 1024, 17, 0, 4.2), (768, 2048, 8, 0, -1.9), (768, 3072, 32, 50000, 43.6),
    (768, 4096, 16, 8000, -5.2), (768, 8192, 17, 20000, 5.8), (768, 8192, 32, 0, -8.2), (1024, 1024, 32, 0, 4.9),
    (1024, 2048, 32, 0, 2.0), (1024, 2048, 1, 0, -2.6), (1024, 3072, 32, 0, 2.1), (1024, 4096, 16, 500, -7.3),
    (1024, 4096, 32, 50000, 49.1), (1024, 8192, 16, 20000, -5.0), (1024, 8192, 32, 500, -9.7),
]


def test_fp32_slices_against_measured_times(rules):
    for d, ff, rows, words, us in FFN2:
        cut = rules.slices(d, ff, rows, (words + 63) // 64 * 4 if words else (3 * d + 15) // 16)
        assert us <= 2.2 if cut else us >= -1.7, (d, ff, rows, words)
    assert not rules.slices(512, 1023, 8, 96) and not rules.slices(512, 1 << 20, 33, 96) and not rules.slices(1025, 1 << 20, 8, 96)
    assert rules.slices(1024, 1 << 30, 32, 1 << 20) and not rules.slices(64, 1024, 32, 1 << 27)


def _matrices(d, ff, gated, n_layer, vocab):
    """Packed weights in the order of their places: (first value, values)."""
    at, out = 0, []
    for _ in range(n_layer):
        for n in (3 * d * d, d * d, (2 if gated else 1) * ff * d, ff * d):
            out.append((at, n))
            at += n
    return out + [(at, (vocab + 63) // 64 * 64 * d)]


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("d,ff", [(768, 3072), (1024, 4096), (2048, 8192), (3072, 8192), (3584, 18944), (4096, 11008), (8192, 28672)])
def test_kept_weights_leave_room_in_the_cache(rules, d, ff, gated):
    for n_layer, vocab in itertools.product((1, 2, 3, 6, 7, 8, 12, 24), (1000, 32000, 50265, 256000)):
        m = _matrices(d, ff, gated, n_layer, vocab)
        kept = [(a, n) for a, n in m if rules.kept(C.c_int64(a), C.c_int64(n))]
        total = 2 * sum(n for _, n in kept)
        assert total <= 210e6                                # of 256 MB, whatever the matrices' sizes
        assert kept == m[:len(kept)]                         # from layer 0 on
        if len(kept) < len(m):                               # until the next one starts or ends too late
            assert total >= 110e6 or total + 2 * m[len(kept)][1] > 210e6


def test_kept_weights_at_the_line(rules):
    assert rules.kept(C.c_int64(0), C.c_int64(105000000)) and not rules.kept(C.c_int64(0), C.c_int64(105000001))
    assert rules.kept(C.c_int64(54999999), C.c_int64(50000001)) and not rules.kept(C.c_int64(54999999), C.c_int64(50000002))
    assert not rules.kept(C.c_int64(55000000), C.c_int64(1))


def test_room_for_row_sums(rules):
    rules.sums.restype = C.c_int64
    for rows, d in itertools.product((16, 32, 64, 80, 112, 128, 256, 4096), (32, 64, 1056, 2048, 8192)):
        room = rules.sums(rows, d)
        assert room >= min(rows, 128) * (d // 16) and room >= 16 * (d // 16) + 16 * (d // 8)
        assert room == max(min(rows, 128), 48) * (d // 16)


def test_words_tell_row_sums_of_half_tiles(rules):
    """... beside the tiles and whether c2 follows c1 (the first bit of the flags)."""
    out = (C.c_int64 * 6)()
    for tiles, flags in itertools.product((1, 192, (1 << 24) + 1, (1 << 30) - 1), (0, 1, 2, 3)):
        rules.words(C.c_int64(64), 2048, 4, tiles, flags, out)
        assert list(out)[1:] == [64, 4, tiles, flags & 1, flags >> 1]


# width, inner width; rows with low parts; on request: 0 norm kernel, 1 whole tiles, 2 halves
HANDOVER = [
    (1024, 512, 1, 0, 1), (1024, 4096, 1, 0, 1), (1024, 4128, 1, 0, 0), (1024, 4128, 1, 1, 1), (1024, 512, 0, 0, 1),
    (1056, 64, 1, 0, 2), (1056, 96, 1, 0, 0), (1056, 96, 1, 1, 1), (1056, 64, 0, 0, 0), (1056, 64, 0, 1, 1), (1536, 6144, 1, 0, 2),
    (1536, 6144, 1, 1, 2), (1536, 6208, 1, 0, 0), (2048, 6144, 1, 0, 2), (2080, 512, 1, 0, 0), (2080, 512, 1, 1, 1), (4096, 11008, 1, 0, 0),
]


@pytest.mark.parametrize("d,ff,low,request_,expect", HANDOVER)
def test_norm_handover_on_both_sides_of_its_lines(rules, d, ff, low, request_, expect):
    assert rules.handover(d, ff, low, request_) == expect


# fp32 attention: head size, units, context keys; us per step of 4 layers with one block per unit and with two
F32_ATTENTION = [
    (64, 8, 160, 122.7, 111.7), (64, 8, 700, 151.7, 135.4), (64, 8, 4000, 343.7, 277.6), (64, 64, 160, 127.6, 117.7),
    (64, 64, 2000, 247.5, 207.5), (64, 128, 160, 180.5, 172.8), (64, 128, 700, 208.7, 197.3), (64, 128, 2000, 307.8, 265.2),
    (64, 160, 160, 181.2, 193.5), (64, 160, 700, 213.3, 238.2), (64, 256, 320, 191.6, 210.4), (64, 256, 700, 238.6, 262.4),
    (32, 8, 320, 109.6, 114.2), (32, 8, 480, 109.1, 112.1), (64, 8, 20, 113.3, 118.4),
    (40, 8, 160, 118.5, 114.2), (40, 128, 700, 189.3, 180.3), (50, 128, 160, 171.3, 174.4), (50, 128, 700, 227.6, 207.2),
    (96, 128, 160, 227.4, 217.4), (128, 8, 160, 163.0, 153.8), (128, 128, 2000, 536.5, 442.2), (200, 4, 700, 355.9, 305.5),
    (256, 64, 160, 296.2, 268.8), (36, 160, 700, 176.1, 218.4),
]


@pytest.mark.parametrize("hd,units,keys,one,two", F32_ATTENTION)
def test_f32_attention_blocks_are_near_the_fastest_measured(rules, hd, units, keys, one, two):
    assert (two if rules.f32_halves(hd, units, keys) else one) <= 1.02 * min(one, two)


def test_f32_attention_blocks_at_the_lines(rules):
    for hd, units, keys, two in ((32, 8, 300, 0), (33, 8, 300, 1), (64, 128, 300, 1), (64, 129, 300, 0), (64, 8, 159, 0), (64, 8, 160, 1)):
        assert rules.f32_halves(hd, units, keys) == two
