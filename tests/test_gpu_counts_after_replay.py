"""Counts after a replayed graph of the caller's: a check reads the device's
counts, but the getters after a further replay report that replay's, not the
check's.  The master slides by parts of an element from replay to replay, so
that candidates, pairs and nonzeros change in number."""

import numpy as np
import pytest
import torch

import synth
from tests.test_gpu_workspace import _iface

pytestmark = pytest.mark.gpu


def getter_outputs(it, which):
    if which == "stats":
        st = it.stats()
        return [st[k] for k in ("n_candidates", "n_pairs", "nnz_D", "nnz_M", "nverts_hist")]
    if which == "refresh":
        it.refresh()
        return [it.n_cand, it.n_pairs, it.nnz_D, it.nnz_M]
    if which == "csr":
        return [t.cpu().numpy() for t in (it.D_rowptr, it.D_col, it.M_rowptr, it.M_col)]
    return [t.cpu().numpy() for t in getattr(it, which)()]


@pytest.mark.parametrize("which", ["stats", "pairs", "candidates", "csr", "refresh"])
def test_getter_after_check_and_replay(which):
    itf = synth.interface_config(2, scale=32)
    h = 1.0 / 32
    it = _iface(itf)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    it.set_capacity()
    with torch.cuda.stream(s):  # warm-up on the capture stream
        it.build_pairs(sync=False)
        it.csr_pattern(sync=False)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        it.build_pairs(sync=False)
        it.csr_pattern(sync=False)
    seen = set()
    for step in range(3):
        # x grows by step * 0.37 of an element: other overlaps, other counts
        moved = itf.master.X + np.array([0.37 * h * step, 0.0, 0.0])
        it.Xm.copy_(torch.from_numpy(moved).t())
        torch.cuda.synchronize()
        print(f"[gpu] replay {step}, then {which}", flush=True)
        g.replay()
        torch.cuda.synchronize()
        if step < 2:
            it.check()
            continue
        fresh = _iface(itf, itf.slave.X, moved).setup()
        seen.add(fresh.n_pairs)
        for a, b in zip(getter_outputs(it, which), getter_outputs(fresh, which)):
            assert np.array_equal(a, b)
    # the replays before it did have other counts
    for step in range(2):
        seen.add(_iface(itf, itf.slave.X, itf.master.X + np.array([0.37 * h * step, 0.0, 0.0])).setup().n_pairs)
    assert len(seen) == 3
