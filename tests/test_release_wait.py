"""The device code as built: every cache write-back and invalidation is waited for before the next
memory access.  An L2 write-back that is still under way when the executor's completion counter is
added to lets a workgroup of another XCD read stale tiles."""
import os
import re
import struct
import subprocess

import pytest

import paper_2009_07482_amd as psc

LLVM = "/opt/rocm/llvm/bin/"
LIB = os.path.join(os.path.dirname(psc.__file__), "libpsc.so")


def _code_objects(path, tmp):
    """The gfx950 code objects of the offload bundles in `path`."""
    fat = os.path.join(tmp, "fat")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section=.hip_fatbin=" + fat, path, os.path.join(tmp, "copy")],
                   check=True)
    with open(fat, "rb") as f:
        data = f.read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n] and size:
                yield data[at + off:at + off + size]
            p += 24 + n
        at += len(magic)


@pytest.mark.skipif(not os.path.exists(LLVM + "llvm-objdump") or not os.path.exists(LIB), reason="no build tools")
def test_cache_operations_are_waited_for(tmp_path):
    seen = 0
    for i, co in enumerate(_code_objects(LIB, str(tmp_path))):
        f = tmp_path / f"co{i}"
        f.write_bytes(co)
        text = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", str(f)], capture_output=True,
                              text=True, check=True).stdout
        lines = [x.split("//")[0].strip() for x in text.splitlines()]
        for k, op in enumerate(lines):
            if not re.match(r"buffer_(wbl2|inv)\b", op):
                continue
            seen += 1
            after = next(x for x in lines[k + 1:] if re.match(r"(global|flat|buffer|scratch|ds)_|s_barrier|s_endpgm", x)
                         or "vmcnt(0)" in x)
            assert "vmcnt(0)" in after, f"{op}: {after} comes before a wait"
    assert seen > 0
