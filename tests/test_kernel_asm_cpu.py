"""Orderings in the compiled kernels that no run would show to be missing (compiled here, no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2103_08053_amd import build


def _kernels(src, tmp_path):
    """Instructions of every kernel of a source file, by mangled name."""
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    out = tmp_path / "a.s"
    subprocess.check_call([hipcc, *build.HIPCC_FLAGS, "-x", "hip", "--cuda-device-only", "-S",
                           os.path.join(build.CSRC, src), "-o", str(out)])
    text = out.read_text()
    return dict(re.findall(r"^(_Z\w+):\s*;[^\n]*\n(.*?)s_endpgm", text, re.M | re.S))


def test_small_count_finishes_its_adds_before_the_last_workgroup_reads_them(tmp_path):
    """The last workgroup halves the per-vertex sums, so each wavefront of every workgroup has to wait for its
    own adds before the barrier that precedes the count of finished workgroups."""
    kernels = {k: v for k, v in _kernels("tc_small.hip", tmp_path).items() if re.search(r"k_small_countILj\d+ELb1E", k)}
    assert len(kernels) == 7
    for name, body in kernels.items():
        parts = body.split("s_barrier")
        assert len(parts) == 4, name  # set-up, the adds, the count of finished workgroups, the finish
        adds = parts[1]
        tail = adds[adds.rindex("global_atomic_add_x2"):]
        assert "s_waitcnt vmcnt(0)" in tail, name
