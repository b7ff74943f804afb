"""The device executor as built: an instance reserves the LDS of the functions it holds, and spills
next to nothing."""
import os
import re
import subprocess

import pytest

from test_release_wait import LIB, LLVM, _code_objects

# groups of tile functions and the LDS of the largest of them: a padded 64 x 64 FP32 transpose tile,
# four 16 x 64 FP32 partial tiles of pitch 68, four wavefronts' staged BF16 columns
LARGEST = {1 << 13: 64 * 65 * 4, 1 << 13 | 7 << 3: 4 * 16 * 68 * 4, 1 << 13 | 7 << 3 | 1: 4 * 16 * 68 * 4,
           1 << 13 | 7 << 10: 4 * 8 * 16 * 40 * 2, 1 << 13 | 7 << 10 | 3 << 6: 4 * 8 * 16 * 40 * 2}
OWN = 64 * 16 + 128 + 16   # the task list, the current kernel, a flag


@pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf") or not os.path.exists(LIB), reason="no build tools")
def test_instances_reserve_what_they_use(tmp_path):
    seen = {}
    for i, co in enumerate(_code_objects(LIB, str(tmp_path))):
        f = tmp_path / f"co{i}"
        f.write_bytes(co)
        notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(f)], capture_output=True, text=True,
                               check=True).stdout
        for block in re.split(r"\n  - (?=\.agpr_count|\.args)", notes):
            name = re.search(r"\.name:\s+\S*exec_kernelILj(\d+)E", block)
            if name:
                seen[int(name.group(1))] = {k: int(re.search(rf"\.{k}:\s+(\d+)", block).group(1))
                                            for k in ("group_segment_fixed_size", "vgpr_spill_count")}
    assert set(LARGEST) <= set(seen), sorted(seen)
    for groups, lds in LARGEST.items():
        assert lds <= seen[groups]["group_segment_fixed_size"] <= lds + OWN, (groups, seen[groups])
    assert all(v["vgpr_spill_count"] <= 4 for v in seen.values()), seen
