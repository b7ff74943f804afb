"""The enqueueing threads over two plans of different stream counts (host only): a native check, with
errors in the middle of runs of either."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_07482_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_two_plans_of_different_stream_counts(tmp_path):
    exe = str(tmp_path / "dispatch_check")
    src = [os.path.join(ROOT, "tests", "native", "dispatch_check.cpp")] + [
        os.path.join(CSRC, f) for f in ("dispatch.cpp", "sched.cpp", "dag.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, *src,
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-500:]
