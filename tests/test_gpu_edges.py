"""Sizes at which a kernel or a dispatch rule changes over, each against the fp64 oracle (bars of tests/measures.py)."""
import numpy as np
import pytest

import oracle
from paper_2605_08123_amd.workloads import Workload, make_inputs
from tests.measures import TOL, assert_per_tensor, floors
from tests.test_gpu_parity import check, rel, run_gpu

pytestmark = pytest.mark.gpu


def work(name, L, d, W, T, dtype, H=1, R=2, **kw):
    return Workload(name, 0, B=1, H=H, L=L, d=d, W=W, T=T, R=R, eps=0.8, dtype=dtype, **kw)


@pytest.mark.parametrize("L", [4094, 4095, 4096, 8190, 8191, 8192, 9000])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_dustbin_element_batches(dtype, L):
    """L + 1 values in batches of 8192 (half-steps) or 4096 (mat-vecs), then single ones."""
    check(work("dustbin_edge", L, 32, 5, 2, dtype, dustbin=True, dustbin_score=0.3))
