"""The prediction that chooses a fine schedule's queue count ends for runs of any length (host only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_07482_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_prediction_ends(tmp_path):
    exe = str(tmp_path / "predict_check")
    src = [os.path.join(ROOT, "tests", "native", "predict_check.cpp")] + [
        os.path.join(CSRC, f) for f in ("group.cpp", "sched.cpp", "dag.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, *src, "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:]
