"""Operators and gradients on both sides of the numbers of slave elements at
which the places of the block rows go to workgroups of their own, against the
oracle (the master side covers a corner of the slave side only, to keep the
oracle's work small)."""

import numpy as np
import pytest

import oracle
from synth.meshes import Interface, Mesh
from tests.gpu_util import TOL, assert_forward_parity, gpu_run, oracle_params, rel_err
from tests.test_gpu_backward import oracle_grad
from tests.test_gpu_search_sizes import patch

pytestmark = pytest.mark.gpu


# slave elements: 163,840 and 164,016
@pytest.mark.parametrize("nx,ny", [(512, 320), (402, 408)])
def test_sizes(nx, ny):
    itf = patch(nx, ny)
    corner = np.nonzero(itf.master.X[itf.master.conn].mean(1)[:, :2].max(1) < 0.12)[0]
    used, conn = np.unique(itf.master.conn[corner], return_inverse=True)
    itf = Interface(itf.slave, Mesh(itf.master.X[used], conn.reshape(-1, 4).astype(np.int32)), itf.delta,
                    name=f"corner of {nx}x{ny}")
    print(f"[gpu] {itf.name}", flush=True)
    prm = oracle_params(itf)
    g = gpu_run(itf, backward_seed=3300)
    o = oracle.evaluate(itf, prm)
    assert len(o["pair_s"]) > 1000
    assert_forward_parity(g, o)
    for k, r in zip(("gXs", "gXm"), oracle_grad(itf, prm, o["pair_s"], o["pair_m"], 3300)):
        assert rel_err(g[k], r) <= TOL, k
