"""The device code as built: a kernel that may run as part of a shared launch reads its argument
record in one go before it branches on the table of shared launches.  A record read behind that
branch costs every launch of one kernel a further memory round trip."""
import os
import re
import subprocess

import pytest

import paper_2009_07482_amd as psc

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
HSACO = os.path.join(os.path.dirname(psc.__file__), "libpsc_kernels.hsaco")
# bytes of pointers and strides at the start of the argument records (kernels.hpp)
HEAD = {"GemmArgs": 48, "SoftmaxArgs": 32, "TransArgs": 32, "AddArgs": 48}


@pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(HSACO), reason="no build tools")
def test_records_are_read_before_the_table_is_looked_at():
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", HSACO], capture_output=True, text=True,
                          check=True).stdout
    seen = 0
    for block in re.split(r"\n(?=[0-9a-f]{16} <)", text):
        head = re.match(r"[0-9a-f]{16} <([^>]+)>:", block)
        args = head and next((a for a in HEAD if a in head.group(1)), None)
        if not args or "_big_kernel" in block[:200] or "_w4_kernel" in block[:200]:   # (never shared)
            continue
        read = set()
        for line in block.splitlines()[1:]:
            op = line.split("//")[0].strip()
            if op.startswith("s_cbranch"):
                break
            load = re.match(r"s_load_dword(?:x(\d+))? \S+, s\[0:1\], (0x[0-9a-f]+)", op)
            if load:
                at = int(load.group(2), 16)
                read.update(range(at, at + 4 * int(load.group(1) or 1)))
        assert read >= set(range(HEAD[args])), f"{head.group(1)}: the record is read behind a branch"
        seen += 1
    assert seen > 50
