"""Launches in which every block takes the transcript step of the round before
(no GPU): the sums they read and the words their blocks store are apart."""
import os
import subprocess

import pytest

from paper_2508_21393_amd import binding as B
from paper_2508_21393_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_merged_launches_store_no_word_that_another_block_reads(tmp_path):
    if not os.path.exists(B.LIB_PATH):
        pytest.skip("libverilora.so not built")
    exe = str(tmp_path / "partials")
    lib = os.path.dirname(B.LIB_PATH)
    r = subprocess.run([build.hipcc()] + build.COMMON + ["-I", build.CSRC, os.path.join(HERE, "native", "partials.cpp"),
                       "-o", exe, "-L", lib, "-lverilora", f"-Wl,-rpath,{lib}", "-pthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stdout + r.stderr
