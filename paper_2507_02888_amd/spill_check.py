"""Vector-register spills placed where no lane is active, in the device assembly of a
build.

The compiler may put the store of a spilled vector register at the start of a block
where lanes join again (a loop's exit above all), ahead of the instruction that brings
them back (s_or_b64 exec, exec, ...).  At a loop's exit the mask is then zero, the store
does nothing, and what is read back later is stale.  Kernels that hold such a place have given
wrong results only now and then, so the build looks for it.
"""
from __future__ import annotations

import re
import sys

_LABEL = re.compile(r"^\.LBB\d+_\d+:|^; %bb")
_KERNEL = re.compile(r"^(_Z\w+):")
_BEFORE = ("v_writelane", "v_readlane", "s_waitcnt", "s_nop", "s_mov")  # what may stand ahead of the store
_STORE = ("scratch_store", "v_accvgpr_write")


def misplaced_spills(lines):
    """[(kernel, instruction)] of the spills ahead of a block's restored mask."""
    found = []
    kernel, block = None, None  # block: the instructions since a block's start, None once it is past the question
    for line in lines:
        if line.startswith((".LBB", "; %bb")) and _LABEL.match(line):
            block = []
            continue
        if line.startswith("_Z"):
            m = _KERNEL.match(line)
            if m:
                kernel, block = m[1], None
            continue
        if kernel is None or block is None:
            continue
        s = line.strip()
        if not s or s[0] in ";.":
            continue
        if s.startswith("s_or_b64 exec, exec"):
            first = next((i for i, x in enumerate(block) if x.startswith(_STORE)), None)
            if first is not None and all(x.startswith(_BEFORE) for x in block[:first]):
                found.append((kernel, block[first]))
            block = None
        elif s.startswith(("s_cbranch", "s_branch", "s_setpc")) or "exec" in s.split(";")[0]:
            block = None
        else:
            block.append(s)
    return found


def main(paths) -> int:
    bad = 0
    for path in paths:
        with open(path) as f:
            for kernel, store in misplaced_spills(f):
                print(f"{path}: {kernel}: {store}")
                bad += 1
    return 1 if bad else 0


if __name__ == "__main__":
    sys.exit(main(sys.argv[1:]))
