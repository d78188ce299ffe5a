"""A small contact zone on a large slave side (500 x 500 elements) with
capacities for its few pairs: the build without a caller workspace takes it,
and everything computed after it, the calls repeated in another order too,
equals the build in a caller workspace bit for bit."""

import ctypes

import numpy as np
import pytest
import torch

from synth.meshes import Interface, Mesh, tensor_grid
from tests.gpu_util import gpu_params
from tests.test_zz_no_alloc import _outputs

pytestmark = pytest.mark.gpu


def patch():
    """Master 12 x 12 over a twentieth of the slave side's length."""
    out = []
    for n, lo, size, z in ((500, 0.0, 1.0, 0.0), (12, 0.31, 0.05, 1e-4)):
        s, t, conn, _ = tensor_grid(n, n)
        x, y = lo + size * s, lo + size * t
        out.append(Mesh(np.stack([x, y, z + 0.01 * np.sin(20 * x) * np.sin(17 * y)], 1), conn))
    return Interface(*out, 1e-3, name="patch of 500x500")


@pytest.mark.parametrize("dual,nodal", [(False, False), (True, True)])
def test_static_build_of_a_patch(dual, nodal):
    from paper_2202_03933_amd import MortarInterface
    from paper_2202_03933_amd import _capi as C
    itf = patch()
    cap = C.mt_capacity(20000, 4000, 4000, 65536)
    its = []
    for static in (True, False):
        print(f"[gpu] {itf.name} dual={dual} nodal={nodal} static={static}", flush=True)
        it = MortarInterface(torch.from_numpy(itf.slave.X), torch.from_numpy(itf.slave.conn),
                             torch.from_numpy(itf.master.X), torch.from_numpy(itf.master.conn),
                             params=gpu_params(itf, dual=dual, nodal=nodal), device=torch.device("cuda", 0))
        if static:
            nc, npairs = ctypes.c_int64(), ctypes.c_int64()
            C.check(C.lib().mt_build_pairs_static(it.h, ctypes.byref(cap), ctypes.byref(nc), ctypes.byref(npairs),
                                                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
            it.n_cand, it.n_pairs = nc.value, npairs.value
        else:
            it.set_capacity(cap)
            it.build_pairs()
        it.csr_pattern()
        its.append(it)
    a, b = its
    assert (a.n_cand, a.n_pairs, a.nnz_D, a.nnz_M) == (b.n_cand, b.n_pairs, b.nnz_D, b.nnz_M) and a.n_pairs > 500
    for x, y in zip(a.candidates() + a.pairs(), b.candidates() + b.pairs()):
        assert torch.equal(x, y)
    first = [tuple(t.clone() for t in _outputs(it)) for it in its]
    assert all(torch.equal(x, y) for x, y in zip(*first))
    a.check()
    # the pattern once more after a reverse sweep, and the sweep before the values
    a.csr_pattern()
    again = _outputs(a)
    assert all(torch.equal(x, y) for x, y in zip(again, first[0]))
