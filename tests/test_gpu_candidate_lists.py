"""Candidate lists of every length around the limits of the fill pass (half
and all of the entries kept per slave element, and past the long lists' LDS
segment), short and long side by side in one wavefront.  Candidates and
vertex counts against the oracle, bit for bit."""

import numpy as np
import pytest

import oracle
from synth.meshes import Interface, Mesh

pytestmark = pytest.mark.gpu


def strips(counts):
    """Slave elements two apart, each over a strip of counts[i] master
    elements (in shuffled order) that overlap its width; the last strip
    element only touches its box."""
    rng = np.random.default_rng(7)
    quad = np.array([[0, 0], [1, 0], [1, 1], [0, 1]], dtype=float)
    sx, mx = [], []
    for i, c in enumerate(counts):
        o = np.array([3.0 * i, 0.0])
        sx.append(np.c_[quad + o, np.zeros(4)])
        h = 1.0 / max(c - 1, 1)
        for k in range(c):
            q = quad * [0.9, 0.98 * h] + o + [0.05, k * h + (1e-4 if k == c - 1 else 0.0)]
            mx.append(np.c_[q, np.full(4, 2e-4)])
    order = rng.permutation(len(mx))
    mx = [mx[i] for i in order]
    conn = lambda n: np.arange(4 * n, dtype=np.int32).reshape(n, 4)
    return Interface(Mesh(np.concatenate(sx), conn(len(sx))), Mesh(np.concatenate(mx), conn(len(mx))), 1e-3,
                     name=f"strips {counts}")


@pytest.mark.parametrize("counts", [(1,), (16,), (17,), (32,), (33,), (1, 15, 16, 17, 31, 32, 33, 48, 49, 2),
                                    tuple([3] * 31 + [32] + [0 + 1] * 40)])
def test_lists(counts):
    from paper_2202_03933_amd import MortarInterface, default_params
    itf = strips(counts)
    print(f"[gpu] {itf.name[:80]}", flush=True)
    it = MortarInterface(itf.slave.X, itf.slave.conn, itf.master.X, itf.master.conn,
                         params=default_params(delta=itf.delta), device="cuda:0").setup()
    cs, cm = oracle.search(itf.slave, itf.master, itf.delta)
    assert np.bincount(cs, minlength=len(counts)).tolist() == list(counts)
    nv, _, _ = oracle.eval_candidates(itf.slave, itf.master, oracle.params(delta=itf.delta), cs, cm, integrate=False)
    for a, b in zip(it.candidates(), (cs, cm, nv)):
        assert np.array_equal(a.cpu().numpy(), b)
