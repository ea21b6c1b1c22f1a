"""Every rung of the design ladder runs Shoup butterflies: the kernels of its
translation unit read (W, W') pairs, none of them the library's own form of the
root powers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJ = os.path.join(ROOT, "paper_2109_14704_amd", "_build", "tr_ladder.o")


@pytest.mark.skipif(not os.path.exists(OBJ) or shutil.which("nm") is None, reason="needs the built objects and nm")
def test_rungs_read_shoup_pairs():
    syms = [l for l in subprocess.check_output(["nm", "-C", OBJ], text=True).splitlines() if "__device_stub__k_" in l]
    kernels = {l.split("__device_stub__")[1].split("(")[0].split("<")[0] for l in syms}
    assert {"k_naive_stage", "k_fwd_simd", "k_ladder_cols", "k_ladder_blocks"} <= kernels
    assert not [l for l in syms if "TwM" in l]
