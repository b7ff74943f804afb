"""The tile of a launch of several GEMMs (host only): a native check, linked with the library, that a
short member does not set the tile of long ones and that the summation order is kept."""
import os
import shutil
import subprocess

import pytest

import paper_2009_07482_amd as psc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.dirname(psc.__file__)
ROCM = "/opt/rocm"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM + "/include/hip"), reason="no build tools")
def test_group_tiles(tmp_path):
    exe = str(tmp_path / "group_tile_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM + "/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "native", "group_tile_check.cpp"), os.path.join(PKG, "libpsc.so"),
                    "-L" + ROCM + "/lib", "-lamdhip64", "-Wl,-rpath," + PKG + ":" + ROCM + "/lib", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-500:]
