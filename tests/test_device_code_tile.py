"""The gfx950 code of the large-tile LM head with 8 to 10, 17 and 18 row tiles and on row-major weights: accumulators beyond the 256 accumulation registers are
vector registers, which the compiler may use for other values too, and operands of the products are written by vector instructions.  Nothing runs on a GPU."""
import os
import re
import shutil
import subprocess

import pytest

from test_device_code import LIB, OBJDUMP, _next, _registers, _wait_states

pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs ROCm's llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(row tiles, loads, nontemporal stores): [(address, instruction, rest of the line)]}"""
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
                m = re.match(r"_ZN5specv(?:19lm_head_tile|23lm_head_rowmajor)_kernelILi(\d+)ELNS_9MfmaLoadsE([0-4])ELb([01])E", head[1])
                code = out.setdefault((int(m[1]), int(m[2]), m[3] == "1"), []) if m else None
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(.*)", line)
            if m and code is not None:
                code.append((int(m[2], 16), m[1].strip(), m[3]))
    assert {k[0] for k in out if k[1] < 3} == {8, 9, 10, 17, 18} and {k[:2] for k in out if k[1] >= 3} == {(tm, kind) for tm in range(8, 17) for kind in (3, 4)}, sorted(out)
    return out


def test_loads_and_stores_are_nontemporal_where_asked_for(kernels):
    for (tm, kind, nt), code in kernels.items():
        stores = [t for _, t, _ in code if t.startswith("global_store_dwordx4")]
        loads = [t for _, t, _ in code if re.match(r"(global|buffer)_load_dwordx4", t)]
        assert stores and loads
        assert all(t.endswith(" nt") == nt for t in stores), (tm, kind, nt)
        assert all(t.endswith(" nt") == (kind in (2, 4)) for t in loads), (tm, kind, nt)
        assert not [t for _, t, _ in code if t.startswith("scratch_")], (tm, kind, nt)


def test_matrix_instructions_keep_their_distance_from_other_accesses_of_their_registers(kernels):
    """On every way through the code: at least 2 wait states between a vector instruction that writes a register and an MFMA that reads it (its
    accumulators included), and at least 20 between an MFMA (8 passes) and any other instruction that touches its accumulators, accumulation or
    vector registers."""
    def both(text):
        return {("v", r) for r in _registers(text, "v")} | {("a", r) for r in _registers(text, "a")}

    checked = 0
    for key, code in kernels.items():
        at = {a: i for i, (a, _, _) in enumerate(code)}
        after = _next(code, at)
        reads, writes, accs = {}, {}, {}
        for i, (_, text, _) in enumerate(code):
            op, _, rest = text.partition(" ")
            if op.startswith("v_mfma"):
                d, a, b, c = rest.split(", ")[:4]
                reads[i], accs[i] = both(a + " " + b + " " + c), both(d)
                assert not accs[i] & both(a + " " + b), (key, text)
                assert both(c) in (accs[i], set()), (key, text)
            elif op.startswith("v_"):
                writes[i] = both(rest if op.startswith("v_swap") else rest.split(",")[0])
        touches = {i: both(t) for i, (_, t, _) in enumerate(code) if i not in accs}

        def walk(start, states, hit):
            todo, seen = [(j, 0) for j in after[start]], {}
            while todo:
                j, waited = todo.pop()
                if waited >= states or seen.get(j, states) <= waited:
                    continue
                seen[j] = waited
                assert not hit(j), (key, code[start], code[j], waited)
                todo.extend((k, waited + _wait_states(code[j][1])) for k in after[j])

        for i, regs in writes.items():
            walk(i, 2, lambda j: j in reads and reads[j] & regs)
        for i, regs in accs.items():
            walk(i, 20, lambda j: j in touches and touches[j] & regs)
        checked += len(accs)
    assert checked > 1000
