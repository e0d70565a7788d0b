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
    """{demangled-ish name: [(address, instruction text)]} of every kernel of the large-tile LM head"""
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
                m = re.match(r"_ZN5specv19lm_head_mfma_kernelILi(\d+)ELb([01])ELb([01])E", head[1])
                code = out.setdefault((int(m[1]), m[2] == "1", m[3] == "1"), []) if m else None
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(.*)", line)
            if m and code is not None:
                code.append((int(m[2], 16), m[1].strip(), m[3]))
    assert len(out) == 32, sorted(out)                     # 9..16 row tiles, nontemporal or not, with block summaries or not
    return out


def test_logits_are_stored_nontemporal_where_asked_for(kernels):
    """The compiler may merge a nontemporal and an ordinary store of the same value; the 16-byte stores of the logits must be what the
    instantiation says."""
    for (tm, nt, summary), code in kernels.items():
        stores = [t for _, t, _ in code if t.startswith("global_store_dwordx4")]
        assert stores
        assert all(t.endswith(" nt") == nt for t in stores), (tm, nt, summary, [t for t in stores if t.endswith(" nt") != nt][:3])
