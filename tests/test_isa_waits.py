"""The direct global->LDS loads are written in inline assembly, where the compiler adds no waits: those that gfx950 asks
for have to stand in the text itself.  Read back from the disassembly of the built library's kernels."""
import glob
import re
import shutil
import subprocess

import pytest

from paper_2606_08804_amd import qdelta

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """[(kernel, [instruction text, ...])] of the library's gfx950 code objects."""
    d = tmp_path_factory.mktemp("code")
    shutil.copy(qdelta.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    out = []
    for obj in sorted(glob.glob(str(d / "*gfx950"))):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", obj], check=True,
                              capture_output=True, text=True).stdout
        for line in text.splitlines():
            head = re.match(r"<(\S+)>:$", line.strip())
            if head:
                out.append((head[1], []))
            elif out and line.startswith("\t"):
                out[-1][1].append(line.split("//")[0].strip())
    return out


def _states(ins):
    """Wait states that an instruction counts for."""
    return int(ins.split()[1], 0) + 1 if ins.startswith("s_nop") else 1


def _direct_loads(kernels):
    n = 0
    for name, code in kernels:
        for i, ins in enumerate(code):
            if "load_lds" in ins:
                n += 1
                yield name, code, i
    assert n > 1000


def test_m0_write_before_direct_load(kernels):
    """One wait state between a scalar write of M0 (the LDS base) and the load that takes it."""
    bad = {name for name, code, i in _direct_loads(kernels) if re.match(r"\S+ m0,", code[i - 1])}
    assert not bad, (len(bad), sorted(bad)[:3])


def _sgprs(operand):
    pair = re.match(r"s\[(\d+):(\d+)\]$", operand)
    if pair:
        return set(range(int(pair[1]), int(pair[2]) + 1))
    one = re.match(r"s(\d+)$", operand)
    return {int(one[1])} if one else set()


def test_vector_write_before_scalar_base(kernels):
    """Five wait states between a vector instruction's write of a scalar register (v_readfirstlane, v_readlane, a
    compare) and a direct load with that register in its base address."""
    bad = {}
    for name, code, i in _direct_loads(kernels):
        base = set().union(*(_sgprs(op.strip(",")) for op in code[i].split()[1:]))
        states, j = 0, i - 1
        while base and j >= 0 and states < 5:
            parts = code[j].split()
            if parts[0].startswith("v_") and len(parts) > 1 and _sgprs(parts[1].strip(",")) & base:
                bad.setdefault(name, []).append((code[j], code[i], states))
                break
            states += _states(code[j])
            j -= 1
    assert not bad, (sum(map(len, bad.values())), sorted(bad), next(iter(bad.values()))[0])
