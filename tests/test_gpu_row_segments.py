"""Rows of M around one, two and four accumulator segments of the assembly
(26 entries each) and past them, single and batched, against the oracle."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_forward_parity, gpu_run, oracle_params
from tests.test_gpu_row_places import strip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [26, 28, 52, 54, 104, 106])
@pytest.mark.parametrize("dual", [False, True])
def test_row_segments(width, dual):
    from paper_2202_03933_amd import MortarBatch
    itf = strip(width // 2 - 1)
    print(f"[gpu] {itf.name} dual={dual}", flush=True)
    o = oracle.evaluate(itf, oracle_params(itf, dual=dual))
    assert np.diff(o["M"].indptr).max() == width
    g = gpu_run(itf, dual=dual)
    assert_forward_parity(g, o)
    D, M, gap = MortarBatch([g["iface"]]).forward()[0]
    assert np.array_equal(D.cpu().numpy(), g["D"].data) and np.array_equal(M.cpu().numpy(), g["M"].data)
    assert np.array_equal(gap.cpu().numpy(), g["g"])
