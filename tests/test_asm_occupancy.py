"""Registers and private memory of the small-batch kernels' generated gfx950 code (no GPU).

No kernel keeps operands in private memory: a conditional select between two
tile offsets once became an indexed load from it, for every operand of the
int8 streaming kernel.  The kernels of 8 waves on one row block are meant to
share a CU three at a time, which takes six waves per SIMD."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2405_03594_amd import build as B


def _kernels(source, tmp_path_factory):
    """name -> (private bytes per lane, waves per SIMD that the registers allow)"""
    if not os.path.exists(B.HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc is not available")
    out = tmp_path_factory.mktemp("asm") / (source + ".s")
    flags = [f for f in B.CFLAGS if f != "-fPIC"]
    r = subprocess.run([B.HIPCC, *flags, "-S", "--cuda-device-only", os.path.join(B.CSRC, source + ".hip"), "-o",
                        str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text, got = out.read_text(), {}
    for m in re.finditer(r"^(_Z\w*\bk_\w+|_Z\w*k_\w+):", text, re.M):
        tail = text[text.index(".Lfunc_end", m.start()):]
        got[m.group(1)] = (int(re.search(r"; ScratchSize: (\d+)", tail).group(1)),
                           int(re.search(r"; Occupancy: (\d+)", tail).group(1)))
    assert got
    return got


@pytest.mark.parametrize("source", ["k_row", "k_wide", "k_int8_quad", "k_int4_quad"])
def test_no_private_memory(source, tmp_path_factory):
    kernels = _kernels(source, tmp_path_factory)
    spilled = {k: v for k, v in kernels.items() if v[0]}
    assert not spilled, spilled
    if source == "k_wide":                             # one row block, up to four staged-row groups, 8 waves
        eight = {k: v for k, v in kernels.items() if re.search(r"k_sparse_wideI.*Li1ELi[1-4]ELi8ELb0E", k)}
        assert len(eight) == 12 and all(v[1] >= 6 for v in eight.values()), eight
    if source == "k_int8_quad":
        eight = {k: v for k, v in kernels.items() if "Li8E" in k}
        assert len(eight) == 2 and all(v[1] >= 6 for v in eight.values()), eight
