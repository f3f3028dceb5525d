"""The direct loads to LDS, which are inline asm: the compiler looks for neither
M0 nor hazards inside it. The sources are read (one definition, M0 named as
written), then attention.hip and gemm.hip are compiled to assembly with the
build's flags and every such load is checked there: M0 written right before it
with one wait state between, M0 touched by nothing else, and no VALU instruction
writing the load's scalar base in the five wait states before it. CPU only."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2412_00408_amd import build

ASM = re.compile(r"asm(?:\s+volatile)?\s*\((.*?)\);", re.S)


def _sources():
    return {f: open(os.path.join(build.CSRC, f)).read() for f in sorted(os.listdir(build.CSRC))
            if f.endswith((".hip", ".hpp"))}


def test_direct_loads_are_defined_once_and_name_m0():
    seen = []
    for f, text in _sources().items():
        for block in ASM.findall(text):
            if "m0" in block.split(":")[0]:
                seen.append((f, "global_load_lds" in block))
                assert re.search(r'"m0"', block), "%s writes M0 without naming it: %s" % (f, block)
    assert seen and all(f == "quake_device.hpp" and lds for f, lds in seen), seen


def _assembly(src):
    flags = [f for f in build.FLAGS if f not in ("-Wall", "-fPIC")]
    cmd = [build.HIPCC, *flags, *build.EXTRA_FLAGS.get(src, []), "--cuda-device-only", "-S", "-o", "-",
           os.path.join(build.CSRC, src)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return [l.split(";")[0].strip() for l in r.stdout.splitlines()]


def _sgprs(op):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", op)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", op)
    return {int(m.group(1))} if m else set()


def _written(ins):
    """Scalar registers the first operand of an instruction names."""
    p = ins.split(None, 1)
    return _sgprs(p[1].split(",")[0].strip()) if len(p) > 1 else set()


def _check(lines):
    code = [l for l in lines if l and not l.startswith(".") and not l.startswith("//")]
    loads = 0
    for i, ins in enumerate(code):
        if not ins.startswith("global_load_lds"):
            assert not re.search(r"\bm0\b", ins) or ins.startswith("s_mov_b32 m0,"), ins
            continue
        loads += 1
        assert re.match(r"s_nop \d+$", code[i - 1]) and code[i - 2].startswith("s_mov_b32 m0,"), \
            code[i - 3:i + 1]
        base = _sgprs(ins.split(",")[-1].split()[0])
        waits, j = 0, i - 1
        while base and waits < 5 and j >= 0:
            p = code[j]
            if not p.endswith(":"):
                if p.startswith("v_"):
                    assert not base & _written(p), (p, ins, code[j:i + 1])
                else:
                    base -= _written(p)   # a scalar instruction wrote it: nothing to wait for
                waits += 1 + (int(p.split()[1]) if p.startswith("s_nop") else 0)
            j -= 1
    return loads


def test_the_check_finds_both_hazards():
    ok = ["v_readfirstlane_b32 s4, v1", "s_mov_b64 s[4:5], s[4:5]", "s_mov_b32 m0, s6", "s_nop 0",
          "global_load_lds_dwordx4 v0, s[4:5]"]
    assert _check(ok) == 1
    with pytest.raises(AssertionError):
        _check([ok[0]] + ok[2:])
    with pytest.raises(AssertionError):
        _check(ok[:3] + ok[4:])
    with pytest.raises(AssertionError):
        _check(ok + ["s_movreld_b32 m0, s2"])


def test_compiled_direct_loads_stand_clear_of_hazards():
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    files = ["attention.hip", "gemm.hip"]
    with ThreadPoolExecutor(2) as ex:
        for f, lines in zip(files, ex.map(_assembly, files)):
            assert _check(lines) >= 100, f
