"""Registers of the fp32 kernels, as the compiler left them in the built library's metadata.  A block of 16 waves has 128 per
lane; what does not fit goes to scratch memory and back in every block, on a path whose launches last a few microseconds.
Projections with one row tile per block (every decode step of at most 32 rows) and attention with wide loads keep
everything in registers, whatever their rows come from; so does attention with scalar loads of pairs in halves of the dims."""

import os
import re
import struct
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_23431_amd", "libpd.so")
READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def device_objects(blob):
    """The gfx950 code objects of a library: bundles of (offset, size, target) entries."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,), p = struct.unpack_from("<Q", blob, at + 24), at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in target:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 24)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Kernel (mangled name) -> bytes of scratch per lane."""
    if not os.path.exists(LIB) or not os.path.exists(READELF):
        pytest.skip("no built library, or no llvm-readelf beside the compiler")
    out, path = {}, tmp_path_factory.mktemp("code") / "object"
    for obj in device_objects(open(LIB, "rb").read()):
        if b"k_lin" not in obj:
            continue
        path.write_bytes(obj)
        notes = subprocess.check_output([READELF, "--notes", str(path)]).decode()
        for kernel in re.split(r"\n  - \.a", notes)[1:]:
            name = re.findall(r"\n    \.name:\s*(\S+)", kernel)[-1]
            out[name] = int(re.search(r"\.private_segment_fixed_size:\s*(\d+)", kernel).group(1))
    return out


def test_projections_of_one_row_tile_use_no_scratch(scratch):
    one = {k: v for k, v in scratch.items() if re.match(r"_Z5k_linI\w+?Li\d+ELi\d+ELi1ELi\d+ELb[01]ELi\d+EE", k)}
    assert len(one) > 100
    assert {k: v for k, v in one.items() if v} == {}


def test_attention_with_wide_loads_uses_no_scratch(scratch):
    wide = {k: v for k, v in scratch.items() if re.match(r"_Z10k_attn_f32I(f|DF16_)Li\d+ELi\d+ELb1E", k)}
    assert len(wide) >= 20
    assert {k: v for k, v in wide.items() if v} == {}


def test_attention_with_scalar_loads_of_pairs_uses_no_scratch_in_halves(scratch):
    halves = {k: v for k, v in scratch.items() if re.match(r"_Z10k_attn_f32IDF16_Li\d+ELi\d+ELb0ELb1ELi2E", k)}
    assert len(halves) >= 3
    assert {k: v for k, v in halves.items() if v} == {}
