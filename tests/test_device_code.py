"""Properties of the gfx950 code of the built library that neither the results nor the source text show.  The device code of
libspecverify.so (built from this tree) is disassembled; nothing runs on a GPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_08151_amd", "libspecverify.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs ROCm's llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(row tiles, loads: 0 buffer, 1 global, 2 nontemporal global, nontemporal stores, block summaries): [(address, instruction, rest of the line)]} of the large-tile LM head"""
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
                m = re.match(r"_ZN5specv19lm_head_mfma_kernelILi(\d+)ELNS_9MfmaLoadsE([012])ELb([01])ELb([01])E", head[1])
                code = out.setdefault((int(m[1]), int(m[2]), m[3] == "1", m[4] == "1"), []) if m else None
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(.*)", line)
            if m and code is not None:
                code.append((int(m[2], 16), m[1].strip(), m[3]))
    # 9..16 row tiles, stores nontemporal or not: buffer loads with and without block summaries, global loads; 11..16: nontemporal loads
    assert len(out) == 48 + 12, sorted(out)
    return out


def test_loads_and_stores_are_nontemporal_where_asked_for(kernels):
    """The compiler may merge a nontemporal and an ordinary store of the same value; the 16-byte stores of the logits, and the loads of
    the weights, must be what the instantiation says."""
    for (tm, kind, nt, summary), code in kernels.items():
        stream = kind == 2
        stores = [t for _, t, _ in code if t.startswith("global_store_dwordx4")]
        loads = [t for _, t, _ in code if re.match(r"(global|buffer)_load_dwordx4", t)]       # (of W; hidden goes to LDS directly)
        assert stores and loads
        assert all(t.endswith(" nt") == nt for t in stores), (tm, nt, summary, [t for t in stores if t.endswith(" nt") != nt][:3])
        assert all(t.endswith(" nt") == stream for t in loads), (tm, stream, summary, [t for t in loads if t.endswith(" nt") != stream][:3])


def _registers(text, kind):
    out = set()
    for a, b in re.findall(r"\b%s\[(\d+):(\d+)\]" % kind, text):
        out |= set(range(int(a), int(b) + 1))
    return out | {int(a) for a in re.findall(r"\b%s(\d+)\b" % kind, text)}


def _next(code, at):
    """indices of the instructions that may follow instruction i, by fall-through and by branch"""
    out = [[] for _ in code]
    base = code[0][0]
    for i, (_, text, tail) in enumerate(code):
        op = text.split()[0]
        target = re.search(r"\+0x([0-9a-f]+)>", tail) if "branch" in op else None
        if "branch" in op and target:
            out[i].append(at[base + int(target[1], 16)])
        if op not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(code):
            out[i].append(i + 1)
    return out


def _wait_states(text):
    return int(text.split()[1], 0) + 1 if text.startswith("s_nop") else 1


def test_matrix_instructions_keep_their_distance_from_other_accesses_of_their_registers(kernels):
    """The MFMAs of the large-tile LM head are assembly statements, for which the compiler inserts no wait states.  On every way through the code:
    at least 2 wait states between a vector instruction that writes a register and an MFMA that reads it, and at least 20 between an MFMA
    (8 passes) and any other instruction that touches its accumulators (the hardware interlocks only MFMAs among themselves)."""
    checked = 0
    for key, code in kernels.items():
        at = {a: i for i, (a, _, _) in enumerate(code)}
        after = _next(code, at)
        reads, writes, accs = {}, {}, {}
        for i, (_, text, _) in enumerate(code):
            op, _, rest = text.partition(" ")
            if op.startswith("v_mfma"):
                d, a, b = rest.split(", ")[:3]
                reads[i], accs[i] = _registers(a + " " + b, "v"), _registers(d, "a")
            elif op.startswith("v_"):
                writes[i] = _registers(rest.split(",")[0], "v")
        touches = {i: _registers(t, "a") for i, (_, t, _) in enumerate(code) if i not in accs}

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
    assert checked > 10000
