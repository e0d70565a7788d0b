"""The gfx950 code of the loads from memory straight to LDS.  They are assembly statements, for which the compiler inserts no wait states: every kernel of the
built library that holds one is disassembled and looked at.  Nothing runs on a GPU."""
import os
import re
import shutil
import subprocess

import pytest

from test_device_code import LIB, OBJDUMP, _next, _registers, _wait_states

pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs ROCm's llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: [(address, instruction, rest of the line)]} of the kernels with loads to LDS"""
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    d = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, stdout=subprocess.DEVNULL)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=d, check=True, capture_output=True, text=True).stdout
        code = None
        for line in text.splitlines():
            head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if head:
                code = out.setdefault(head[1], [])
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(.*)", line)
            if m and code is not None:
                code.append((int(m[2], 16), m[1].strip(), m[3]))
    out = {k: c for k, c in out.items() if any("_load_lds_" in t for _, t, _ in c)}
    for name in ("verify_attn_kernel", "verify_attn_rows_kernel", "lm_head_mfma_kernel", "lm_head_tile_kernel", "lm_head_rowmajor_kernel", "lm_head_big_kernel"):
        assert any(name in k for k in out), name
    return out


def test_loads_to_lds_keep_their_distance_from_the_writes_of_their_scalar_operands(kernels):
    """On every way through the code: at least 1 wait state between a scalar instruction that writes M0, the LDS address, and a load that reads it (the
    hardware does not interlock it: the load would go to the address of the one before), and at least 5 between a vector instruction that writes a scalar register
    and a load that reads that register, as M0 or as its base."""
    checked = 0
    for key, code in kernels.items():
        at = {a: i for i, (a, _, _) in enumerate(code)}
        after = _next(code, at)
        reads = {}
        for i, (_, text, _) in enumerate(code):
            if "_load_lds_" in text:
                reads[i] = {"m0"} | {("s", r) for r in _registers(text, "s")}
        for i, (_, text, _) in enumerate(code):
            op, _, rest = text.partition(" ")
            operands = rest.split(", ")
            if op.startswith("s_"):
                regs, states = {"m0"} if operands[0] == "m0" else set(), 1
            elif op.startswith("v_"):
                # (the second operand: carries and the like)
                regs, states = {("s", r) for r in _registers(" ".join(operands[:2] if "_co_" in op or "_div_scale" in op or "_mad_" in op else operands[:1]), "s")}, 5
                if operands[0] == "m0":
                    regs.add("m0")
            else:
                continue
            todo, seen = [(j, 0) for j in after[i]] if regs else [], {}
            while todo:
                j, waited = todo.pop()
                if waited >= states or seen.get(j, states) <= waited:
                    continue
                seen[j] = waited
                assert not reads.get(j, set()) & regs, (key, code[i], code[j], waited)
                todo.extend((k, waited + _wait_states(code[j][1])) for k in after[j])
        checked += len(reads)
    assert checked > 10000
