import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as _oracle
    _oracle.build()
    return _oracle


# What spec_set_tuning's keys are when nobody has set them: a test that leaves another value behind would take later ones to other kernels.
TUNING_DEFAULTS = {"attn_chunk": 0, "lm_kernel": 0, "lm_big_waves": 8, "attn_plan": 0, "attn_plan_waves": 0, "attn_nr3_waves": 8, "attn_rows_ring": 0, "accept_filter": 0,
                   "attn_rows": 0, "lm_packed_wide": 0, "lm_packed_tile": 0, "lm_mfma_nt": 0, "lm_mfma_rows": 0, "lm_packed_waves": 0}


@pytest.fixture(autouse=True)
def _tuning_defaults(request):
    if request.node.get_closest_marker("gpu"):
        from paper_2605_08151_amd import binding
        for key, value in TUNING_DEFAULTS.items():
            binding.spec_set_tuning(key, value)
