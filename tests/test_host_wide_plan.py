"""Which groups of a call sum their first rounds across the GPU (no GPU)."""
import os
import subprocess

import pytest

from paper_2508_21393_amd import binding as B
from paper_2508_21393_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_first_sweeps_fit_the_gpu(tmp_path):
    if not os.path.exists(B.LIB_PATH):
        pytest.skip("libverilora.so not built")
    exe = str(tmp_path / "plan")
    lib = os.path.dirname(B.LIB_PATH)
    r = subprocess.run([build.hipcc()] + build.COMMON + ["-I", build.CSRC, os.path.join(HERE, "native", "wide_plan.cpp"),
                       "-o", exe, "-L", lib, "-lverilora", f"-Wl,-rpath,{lib}", "-pthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
