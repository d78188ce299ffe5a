"""GPU parity where a slave element's pairs span several tiles of 64 pairs
(the quantities summed per slave element then come in parts): coarse slave
elements over a fine master, and pair counts around whole tiles, against the
oracle in every mode, single and batched."""

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import TOL, assert_forward_parity, csr_weights, gpu_run, oracle_params, rel_err
from tests.test_gpu_normals import oracle_total_grad
from tests.test_gpu_backward import oracle_grad

pytestmark = pytest.mark.gpu

# (slave, master): one element with exactly one tile of 64 pairs; four with 36
# each; nine with 196 to 225 (four or five tiles); 25 with 100 to 121
SIZES = [(1, 8), (2, 11), (3, 41), (5, 48)]


@pytest.mark.parametrize("ns,nm", SIZES)
@pytest.mark.parametrize("dual,nodal", [(False, False), (True, False), (False, True), (True, True)])
def test_coarse_slave(ns, nm, dual, nodal):
    # (boxes of coarse elements over a curved surface: a wide search distance)
    itf = synth.wavy(ns, nm, amp=0.01, delta=0.05)
    prm = oracle_params(itf, dual=dual, nodal=nodal)
    g = gpu_run(itf, dual=dual, nodal=nodal, backward_seed=3300)
    o = oracle.evaluate(itf, prm)
    assert_forward_parity(g, o)
    ref = (oracle_total_grad if nodal else oracle_grad)(itf, prm, o["pair_s"], o["pair_m"], 3300)
    for k, r in zip(("gXs", "gXm"), ref):
        assert rel_err(g[k], r) <= TOL, k


@pytest.mark.parametrize("dual", [False, True])
def test_coarse_slave_elements_and_batch(dual):
    from paper_2202_03933_amd import MortarBatch
    itfs = [synth.wavy(ns, nm, amp=0.01, delta=0.05) for ns, nm in SIZES]
    for itf in itfs[2:]:
        g = gpu_run(itf, dual=dual, element_rule=8)
        o = oracle.evaluate_elements(itf, 8, oracle_params(itf, dual=dual))
        for k in ("D", "M"):
            assert rel_err(g[k].data, o[k].data) <= TOL
        assert rel_err(g["g"], o["g"]) <= TOL
    runs = [gpu_run(itf, dual=dual, backward_seed=3300) for itf in itfs]
    # a bucket that is no whole number of tiles is rounded up to one
    b = MortarBatch([r["iface"] for r in runs], tuning={"bucket": 100, "block": 128})
    W = []
    for itf, r in zip(itfs, runs):
        W.append(tuple(torch.from_numpy(x).to("cuda:0") for x in csr_weights(r["D"], r["M"], itf.slave.n_nodes, 3300)))
    outs = b.forward()
    grads = b.backward(W)
    torch.cuda.synchronize()
    for r, (D, M, gap), (gs, gm) in zip(runs, outs, grads):
        assert np.array_equal(D.cpu().numpy(), r["D"].data) and np.array_equal(M.cpu().numpy(), r["M"].data)
        assert np.array_equal(gap.cpu().numpy(), r["g"])
        assert np.array_equal(gs.cpu().numpy().T, r["gXs"]) and np.array_equal(gm.cpu().numpy().T, r["gXm"])
