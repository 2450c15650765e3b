"""The hand-written LDS reads of the bf16 products, checked in the code that hipcc makes of them: a
register that such a read fills is neither read nor written before a wait for all LDS operations
(the compiler takes the output of inline assembly as written at once)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_19925_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _vgprs(operand):
    m = re.match(r"v\[(\d+):(\d+)\]|v(\d+)\b", operand.strip())
    if not m:
        return range(0)
    lo, hi = int(m.group(1) or m.group(3)), int(m.group(2) or m.group(3))
    return range(lo, hi + 1)


def early_uses(lines):
    """(kernel, instruction) of uses of a register whose hand-written read may still be in flight, in
    the order of the text (a loop's back edge leads to a phase, which begins with its wait)."""
    kernel, in_asm, flying, found, reads = "", False, set(), [], 0
    for line in lines:
        s = line.strip()
        m = re.match(r"(_Z\w+):", s)
        if m:
            kernel, flying = m.group(1), set()
        elif s == ";;#ASMSTART":
            in_asm = True
        elif s == ";;#ASMEND":
            in_asm = False
        elif s.startswith("s_waitcnt") and "lgkmcnt(0)" in s or s.startswith("s_endpgm"):
            flying = set()
        else:
            m = re.match(r"((?:v|ds|global|flat|buffer)_\w+) (.*)", s)
            if m:
                ops = m.group(2).split(", ")
                if in_asm and m.group(1).startswith("ds_read"):
                    reads += 1
                    if flying.intersection(_vgprs(ops[1])):
                        found.append((kernel, s))
                    flying.update(_vgprs(ops[0]))
                elif any(flying.intersection(_vgprs(o)) for o in ops):
                    found.append((kernel, s))
    return found, reads


@pytest.mark.skipif(not shutil.which(HIPCC), reason="needs hipcc")
def test_no_register_is_used_before_its_read_has_landed(tmp_path):
    out = str(tmp_path / "gemm.s")
    flags = [x for x in build.FLAGS if x not in ("-shared",)]
    subprocess.run([HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm.hip"), "-o", out],
                   check=True, stderr=subprocess.DEVNULL)
    found, reads = early_uses(open(out).read().splitlines())
    assert reads > 100
    assert not found, found[:5]
