"""The kernel names bench.py keys its traffic table by: no two kernels of one run share a name, and the names it looks up are kernels of the
library (the mangled symbols of the built library are read, nothing runs)."""
import os
import re

import bench

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "libspecverify.so")


def test_kernels_of_one_run_have_names_of_their_own():
    run = ["void specv::lm_head_packed_kernel<10, 1, 8, true, 2, false, true, false>(unsigned short const*, int)",
           "void specv::lm_head_packed_kernel<10, 1, 8, true, 2, false, true, true>(unsigned short const*, int)",
           "void specv::accept_bonus_kernel<false, true>(specv::DecideArgs, specv::AcceptWorkspace, bool)",
           "void specv::accept_bonus_kernel<false, false>(specv::DecideArgs, specv::AcceptWorkspace, bool)",
           "void specv::lm_head_mfma_kernel<12, (specv::MfmaLoads)1, true, false>(unsigned short const*)", "specv::accept_decide_kernel(specv::DecideArgs)"]
    names = [bench.short_kernel_name(k) for k in run]
    assert names == ["lm_head_packed_kernel", "lm_head_packed_kernel(row-major)", "accept_bonus_kernel(exponentials)", "accept_bonus_kernel(residual)",
                     "lm_head_mfma_kernel", "accept_decide_kernel"]
    assert bench.instantiation(run[4]) == "specv::lm_head_mfma_kernel<12, 1, true, false>"


def test_kernels_that_carry_a_call_exist():
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    symbols = set(re.findall(rb"_ZN5specv\d+([a-z_0-9]+_kernel)", open(LIB, "rb").read()))
    for names in bench.KERNEL_OF_CALL.values():
        for name in names:
            assert name.split("(")[0].encode() in symbols, name
    for name in bench._algorithmic_by_kernel("mid"):
        assert name.split("(")[0].encode() in symbols, name
