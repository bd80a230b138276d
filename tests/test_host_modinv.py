"""The inversion by division steps on the host build (no GPU)."""
import os
import subprocess

from paper_2508_21393_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_running_inverses_stay_in_range(tmp_path):
    exe = str(tmp_path / "modinv")
    r = subprocess.run([build.hipcc()] + build.COMMON + ["-I", build.CSRC, os.path.join(HERE, "native", "modinv.cpp"),
                                                         "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
