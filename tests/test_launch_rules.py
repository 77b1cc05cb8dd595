"""The rules by which launches are shaped (csrc/launch_rules.h), compiled by the host compiler alone: against times measured
for every shape a rule chooses from, and against exhaustive search where the rule is an optimum of its own estimate."""

import ctypes as C
import itertools
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_23431_amd", "csrc")

SOURCE = r"""
#include "launch_rules.h"
extern "C" {
void attn(int hd, int units, int nblk, int cap, int decode, int pair, int streamed, int *out) {
  const AttnShape s = attn_shape(hd, units, nblk, cap, decode, pair, streamed);
  out[0] = s.splits; out[1] = s.waves;
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
