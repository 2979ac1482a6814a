"""The FP64 panel kernels' waits, in the gfx950 assembly of the source (no GPU): a
panel's first stores go to rows that other wavefronts of the block have loaded, so
a barrier behind a wait for every load must come before them."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _waits(body):
    """A wait for all loads right before a barrier, between the first load and the first store."""
    prev, loads = "", False
    for line in body.splitlines():
        ins = line.split(";")[0].strip()
        if not ins or ins.startswith("."):
            continue
        if ins.startswith("global_store"):
            return False
        if loads and ins.startswith("s_barrier") and re.match(r"s_waitcnt.*vmcnt\(0\)", prev):
            return True
        loads |= ins.startswith("global_load")
        prev = ins
    return False


def test_panel_kernels_wait_for_their_loads_before_the_first_store(tmp_path):
    from paper_2502_16555_amd import build as B
    if not shutil.which(B.HIPCC):
        pytest.skip("no HIP compiler")
    out = tmp_path / "panel.s"
    subprocess.run([B.HIPCC, "-x", "hip"] + B.COMMON + B.DEVICE + ["-S", "--offload-device-only",
                   os.path.join(B.CSRC, "kernels_panel.hip"), "-o", str(out)], check=True, capture_output=True)
    kernels = re.findall(r"^(_Z\w*k_panel_(?:reg|tall)\w*):(.*?)^\s*s_endpgm", out.read_text(), re.S | re.M)
    assert len(kernels) == 5
    for name, body in kernels:
        assert _waits(body), name
