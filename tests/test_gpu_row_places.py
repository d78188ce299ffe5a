"""Rows on both sides of the 256 columns up to which the places of the local
block entries are kept as bytes: M rows of one slave element over a strip of
masters, D rows of a node with a fan of slave elements.  Operators and
gradients against the oracle, standard and dual, single and batched."""

import numpy as np
import pytest
import torch

import oracle
from synth.meshes import Interface, Mesh, tensor_grid
from tests.gpu_util import TOL, assert_forward_parity, csr_weights, gpu_run, oracle_params, rel_err
from tests.test_gpu_backward import oracle_grad

pytestmark = pytest.mark.gpu


def grid(nx, ny, lo, hi, z):
    s, t, conn, _ = tensor_grid(nx, ny)
    return Mesh(np.stack([lo[0] + s * (hi[0] - lo[0]), lo[1] + t * (hi[1] - lo[1]), z + 0.0 * s], 1), conn)


def strip(m):
    """One slave element over m masters: M rows of 2 (m + 1) columns."""
    return Interface(grid(1, 1, (0, 0), (1, 1), 0.0), grid(m, 1, (-0.001, -0.001), (1.001, 1.001), 1e-3), 0.01,
                     name=f"strip {m}")


def fan(k):
    """k slave elements around a node: its D row has 2 k + 1 columns."""
    t = 2 * np.pi * np.arange(2 * k) / (2 * k)
    r = np.where(np.arange(2 * k) % 2 == 0, 1.0, 1.05)
    X = np.concatenate([np.zeros((1, 3)), np.stack([r * np.cos(t), r * np.sin(t), 0.02 * r**2], 1)])
    i = np.arange(k)
    conn = np.stack([0 * i, 1 + 2 * i, 2 + 2 * i, 1 + (2 * i + 2) % (2 * k)], 1).astype(np.int32)
    return Interface(Mesh(X, conn), grid(3, 3, (-1.2, -1.1), (1.1, 1.2), 0.01), 0.05, name=f"fan {k}")


CASES = [(strip, 127, 256), (strip, 128, 258), (fan, 127, 255), (fan, 128, 257)]


@pytest.mark.parametrize("dual", [False, True])
@pytest.mark.parametrize("make,k,width", CASES)
def test_row_places(make, k, width, dual):
    from paper_2202_03933_amd import MortarBatch
    itf = make(k)
    print(f"[gpu] {itf.name} dual={dual}", flush=True)
    prm = oracle_params(itf, dual=dual)
    o = oracle.evaluate(itf, prm)
    assert np.diff(o["M" if make is strip else "D"].indptr).max() == width
    g = gpu_run(itf, dual=dual, backward_seed=3300)
    assert_forward_parity(g, o)
    for name, r in zip(("gXs", "gXm"), oracle_grad(itf, prm, o["pair_s"], o["pair_m"], 3300)):
        assert rel_err(g[name], r) <= TOL, name
    W = tuple(torch.from_numpy(x).to("cuda:0") for x in csr_weights(g["D"], g["M"], itf.slave.n_nodes, 3300))
    b = MortarBatch([g["iface"]])
    (D, M, gap), (gs, gm) = b.forward()[0], b.backward([W])[0]
    assert np.array_equal(D.cpu().numpy(), g["D"].data) and np.array_equal(M.cpu().numpy(), g["M"].data)
    assert np.array_equal(gs.cpu().numpy().T, g["gXs"]) and np.array_equal(gm.cpu().numpy().T, g["gXm"])
