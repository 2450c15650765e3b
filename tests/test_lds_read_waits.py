"""The hand-written LDS reads and direct-to-LDS loads of the bf16 products, checked in the code that
hipcc makes of them: a register that such a read fills is neither read nor written before a wait for
all LDS operations (the compiler takes the output of inline assembly as written at once), and a
write of M0 is followed by its wait state before a load that takes its LDS address from M0 (the compiler
puts none into inline assembly)."""
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


def m0_without_wait(lines):
    """(kernel, instruction) of direct-to-LDS loads that directly follow a write of M0."""
    kernel, before, found, loads = "", "", [], 0
    for line in lines:
        s = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):", s)
        if m:
            kernel = m.group(1)
        if not re.match(r"[a-z]+_\w+( |$)", s):   # labels, directives, comments
            continue
        if s.startswith("global_load_lds") or s.startswith("buffer_load") and s.endswith("lds"):
            loads += 1
            if re.match(r"s_\w+ m0,", before):
                found.append((kernel, s))
        before = s
    return found, loads


def _device_code(source, tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("needs hipcc")
    out = str(tmp_path_factory.mktemp("code") / (source + ".s"))
    flags = [x for x in build.FLAGS if x not in ("-shared",)]
    subprocess.run([HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", out],
                   check=True, stderr=subprocess.DEVNULL)
    return open(out).read().splitlines()


@pytest.fixture(scope="module")
def gemm_code(tmp_path_factory):
    return _device_code("gemm.hip", tmp_path_factory)


def test_no_register_is_used_before_its_read_has_landed(gemm_code):
    found, reads = early_uses(gemm_code)
    assert reads > 100
    assert not found, found[:5]


def test_every_m0_write_has_its_wait_state(gemm_code, tmp_path_factory):
    for code in (gemm_code, _device_code("ceilings.hip", tmp_path_factory)):
        found, loads = m0_without_wait(code)
        assert loads > 30
        assert not found, (len(found), found[:5])
