"""GPU search at the sizes where its scans and bins change form: one tile
(2,048 values), the last and first size past a launch whose workgroups add up
the values before them (32 tiles), and every master in one cell.  Candidates,
pairs, vertex counts and row pointers against the oracle, bit for bit."""

import numpy as np
import pytest

import oracle
import synth
from synth.meshes import Interface, Mesh, tensor_grid

pytestmark = pytest.mark.gpu


def patch(nx, ny):
    """nx x ny slave elements under a shifted, rotated and raised master grid
    of about 0.8 times the resolution."""
    h = 1.0 / max(nx, ny)
    sides = []
    for i, (a, b) in enumerate(((nx, ny), (max(1, int(0.8 * nx)), max(1, int(0.8 * ny))))):
        s, t, conn, _ = tensor_grid(a, b)
        x, y = s * nx * h, t * ny * h
        if i:
            x, y = x + 0.03 * y + 0.013, y - 0.03 * x + 0.007
        sides.append(Mesh(np.stack([x, y, 5e-4 * i + 0.01 * np.sin(3 * x) * np.cos(2 * y)], 1), conn))
    return Interface(sides[0], sides[1], 1e-3, name=f"patch {nx}x{ny}")


@pytest.mark.parametrize("nx,ny,bin_size", [(1, 1, 0.0), (89, 23, 0.0), (64, 32, 0.0), (683, 3, 0.0), (257, 255, 0.0),
                                            (256, 256, 0.0), (331, 198, 0.0), (40, 30, 10.0)])
def test_search(nx, ny, bin_size):
    from paper_2202_03933_amd import MortarInterface, default_params
    itf = patch(nx, ny)
    print(f"[gpu] {itf.name} bin_size={bin_size}", flush=True)
    it = MortarInterface(itf.slave.X, itf.slave.conn, itf.master.X, itf.master.conn,
                         params=default_params(delta=itf.delta, bin_size=bin_size), device="cuda:0").setup()
    prm = oracle.params(delta=itf.delta)
    cs, cm = oracle.search(itf.slave, itf.master, itf.delta)
    nv, _, _ = oracle.eval_candidates(itf.slave, itf.master, prm, cs, cm, integrate=False)
    for a, b in zip(it.candidates(), (cs, cm, nv)):
        assert np.array_equal(a.cpu().numpy(), b)
    keep = nv >= 3
    ps, pm = cs[keep], cm[keep]
    for a, b in zip(it.pairs(), (ps, pm, nv[keep])):
        assert np.array_equal(a.cpu().numpy(), b)
    n = itf.slave.n_nodes
    for rowptr, cols, width in ((it.D_rowptr, itf.slave.conn[ps], n), (it.M_rowptr, itf.master.conn[pm],
                                                                       itf.master.n_nodes)):
        keys = np.unique(itf.slave.conn[ps].astype(np.int64)[:, :, None] * width + cols[:, None, :])
        assert np.array_equal(rowptr.cpu().numpy(), np.searchsorted(keys, np.arange(n + 1) * width))
