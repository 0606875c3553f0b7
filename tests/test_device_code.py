"""What the compiled device code has to hold and no result shows (CPU only: the
sources are compiled to assembly, nothing runs)."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from paper_2208_00184_amd import build as hip_build

CSRC = os.path.join(os.path.dirname(hip_build.__file__), "csrc")


def kernels(source, tmp_path):
    """The assembly of every kernel of a source, by mangled name."""
    if not shutil.which("hipcc"):
        pytest.skip("needs hipcc")
    out = str(tmp_path / "device.s")
    subprocess.run(["hipcc", *hip_build.FLAGS, "--offload-device-only", "-S", os.path.join(CSRC, source), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    return {m[1]: m[2] for m in re.finditer(r"^(_Z\w+):.*?\n(.*?)^\.Lfunc_end", text, re.M | re.S)}


def test_blocks_wait_for_their_stores(tmp_path):
    """k_ms_blocks reads finish times that other waves stored two blocks
    before: in every variant one barrier of the loop comes right behind a wait
    for the wave's own vector stores (vmcnt(0)), whatever the wave did before."""
    ks = {k: v for k, v in kernels("ms_blocks.hip", tmp_path).items() if "k_ms_blocks" in k}
    assert len(ks) == 3
    for name, code in ks.items():
        assert re.search(r"s_waitcnt [^\n]*vmcnt\(0\)[^\n]*\n\s*s_barrier", code), name
