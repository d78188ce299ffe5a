"""The CSR arrays copied out into aligned and unaligned buffers, and the
counts read back with them, against the oracle's pattern."""

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nm", [(1, 1), (2, 1), (5, 4), (60, 49), (300, 233)])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_csr_copy(ns, nm, shift):
    from paper_2202_03933_amd import MortarInterface, default_params
    from paper_2202_03933_amd import _capi as C
    itf = synth.wavy(ns, nm, delta=0.05 if ns < 5 else 1.25e-3)
    it = MortarInterface(itf.slave.X, itf.slave.conn, itf.master.X, itf.master.conn,
                         params=default_params(delta=itf.delta), device="cuda:0").setup()
    cs, cm = oracle.search(itf.slave, itf.master, itf.delta)
    nv, _, _ = oracle.eval_candidates(itf.slave, itf.master, oracle_params(itf), cs, cm, integrate=False)
    ps, pm = cs[nv >= 3], cm[nv >= 3]
    n = itf.slave.n_nodes
    want = []
    for cols, width in ((itf.slave.conn[ps], n), (itf.master.conn[pm], itf.master.n_nodes)):
        keys = np.unique(itf.slave.conn[ps].astype(np.int64)[:, :, None] * width + cols[:, None, :])
        want += [np.searchsorted(keys, np.arange(n + 1) * width), keys % width]
    assert (it.nnz_D, it.nnz_M) == (len(want[1]), len(want[3]))
    out = [torch.full((len(w) + shift + 5,), -1, dtype=torch.int32, device="cuda:0") for w in want]
    ptr = [t[shift:].data_ptr() for t in out]
    C.check(C.lib().mt_get_csr(it.h, *ptr, torch.cuda.current_stream().cuda_stream))
    for t, w in zip(out, want):
        t = t.cpu().numpy()
        assert np.array_equal(t[shift:shift + len(w)], w)
        assert (t[:shift] == -1).all() and (t[shift + len(w):] == -1).all()
