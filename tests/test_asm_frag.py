"""The counted waits of the decoded-fragment product (k_gemm.hip), checked on
the generated gfx950 code (no GPU).

At the barrier of a stage a wave has waited until at most XG + 3 FN of its
requests remain, which covers stage st + 1's activations only if, between two
barriers, a wave issues XG LDS requests and 2 FN fragment loads, the last FN of
them after every LDS request.  The source fixes that order with scheduling
fences; this test reads it off each kernel's loop."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2405_03594_amd import build as B


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(B.HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc is not available")
    out = tmp_path_factory.mktemp("asm") / "k_gemm.s"
    flags = [f for f in B.CFLAGS if f != "-fPIC"]
    r = subprocess.run([B.HIPCC, *flags, "-S", "--cuda-device-only", os.path.join(B.CSRC, "k_gemm.hip"), "-o",
                        str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out.read_text()


def test_requests_between_barriers(asm):
    seen = 0
    for m in re.finditer(r"^(_Z\w*k_frag_gemmI\w*?Li(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E\w*):", asm, re.M):
        FN, FM, NWN, NWM = (int(x) for x in m.groups()[1:])
        XG = 16 * FM * NWM // 8 // (NWN * NWM)
        body = asm[m.start():asm.index(".Lfunc_end", m.start())]
        loops = [b for b in re.split(r"\n(?=\.LBB)", body) if len(re.findall("v_mfma", b)) == 8 * FN * FM]
        assert len(loops) == 1, (m.group(1), "the loop is one block of four stages")
        ops, waits = [], []
        for line in loops[0].split("\n"):
            op = line.split()[0] if line.split() else ""
            if op.startswith("buffer_load"):
                ops.append("lds" if line.rstrip().endswith("lds") else "reg")
            elif op == "s_waitcnt" and "vmcnt" in line:
                waits.append(int(re.search(r"vmcnt\((\d+)\)", line).group(1)))
            elif op == "s_barrier":
                ops.append("|")
                assert waits[-1] <= XG + 3 * FN, m.group(1)
        assert ops.count("|") == 4, m.group(1)
        i = ops.index("|")
        for seg in "".join({"lds": "L", "reg": "r", "|": "|"}[o] for o in ops[i + 1:] + ops[:i]).split("|"):
            assert seg.count("L") == XG and seg.count("r") == 2 * FN, (m.group(1), seg)
            assert seg.endswith("r" * FN), (m.group(1), seg)
        seen += 1
    assert seen >= 15
