import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def gemm_plan():
    """ded::bf16_gemm_plan(sum_rows, rows_pad, N, K, planes, max_splits, part_elems): which kernel runs a projection (host code)."""
    import ctypes as C

    from paper_2407_12021_amd import binding

    class Plan(C.Structure):
        _fields_ = [(n, C.c_int) for n in ("nwn", "nw", "splits", "tile", "whole", "ssq_waves")]

    def plan(*args):
        f = binding.lib()["_ZN3ded14bf16_gemm_planEiiiiiil"]
        f.restype, f.argtypes = Plan, [C.c_int] * 6 + [C.c_int64]
        return f(*args)

    return plan


@pytest.fixture(scope="session")
def small_cfg():
    from ded_inputs import ModelConfig
    return ModelConfig("pin-small", 2, 32, 4, 2, 8, 48, 50, dtype="fp32")


@pytest.fixture(scope="session")
def small_model(small_cfg):
    from ded_inputs import make_weights
    # std 0.3 keeps the soft-max far from uniform so that masking / ordering mistakes show up
    return make_weights(small_cfg, seed=3, gain_jitter=0.1, std=0.3)
