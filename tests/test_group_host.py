"""Launch groups of the fine schedules (csrc/group.cpp) on the CPU: a native check over random DAGs,
mappers and copy options that every precedence of the DAG is enforced by the grouped structure and
that nothing is lost, added or grouped against the rules."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_07482_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_launch_groups_keep_every_precedence(tmp_path):
    exe = str(tmp_path / "group_check")
    src = [os.path.join(ROOT, "tests", "native", "group_check.cpp")] + [
        os.path.join(CSRC, f) for f in ("group.cpp", "sched.cpp", "dag.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, *src, "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
