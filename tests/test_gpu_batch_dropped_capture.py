"""A first batch backward recorded in a capture that is dropped and never runs
(recorded with the null pointers that a new build's table holds, so that the
table need not be uploaded): the eager backward after it has every index it
needs.  Instances on the caller's stream alone, whose pattern leaves the
pairs-by-master index and the master incidence to the batch."""

import ctypes

import pytest
import torch

import synth
from tests.gpu_util import gpu_params
from tests.test_gpu_batch import equal_outs, make_ifaces, weights_for

pytestmark = pytest.mark.gpu

THREAD_LOCAL = 1  # hipStreamCaptureModeThreadLocal


@pytest.mark.parametrize("search", [False, True])
def test_backward_after_a_dropped_capture(search):
    from paper_2202_03933_amd import MortarBatch, MortarInterface
    from paper_2202_03933_amd import _capi as C
    from paper_2202_03933_amd.batch import _ptr_table
    instances = synth.batched_instances(n_inst=4, max_side=32)
    refs = make_ifaces(instances)
    W = [weights_for(r, 4500 + k) for k, r in enumerate(refs)]
    ref_g = [tuple(t.clone() for t in r.backward(*w)) for r, w in zip(refs, W)]
    ifaces = []
    for itf in instances:
        p = gpu_params(itf)
        p.single_stream = 1
        ifaces.append(MortarInterface(torch.from_numpy(itf.slave.X), torch.from_numpy(itf.slave.conn),
                                      torch.from_numpy(itf.master.X), torch.from_numpy(itf.master.conn),
                                      params=p, device=torch.device("cuda", 0)).setup())
    b = MortarBatch(ifaces)
    if search:
        b.search(use_graph=True)
    g = [(torch.zeros_like(a), torch.zeros_like(c)) for a, c in ref_g]
    tabs = [_ptr_table([x[k] for x in W]) for k in range(3)] + [_ptr_table([o[k] for o in g]) for k in range(2)]
    torch.cuda.synchronize()
    L = C.lib()
    print(f"[gpu] batch backward in a capture that is dropped, search={search}", flush=True)
    null = (ctypes.c_void_p * len(ifaces))()
    graph = ctypes.c_void_p()
    assert L.hipStreamBeginCapture(b._s(), THREAD_LOCAL) == 0
    rc = L.mt_batch_backward(b.h, null, null, null, null, null, 0, b._s())
    assert L.hipStreamEndCapture(b._s(), ctypes.byref(graph)) == 0 and rc == C.MT_OK
    assert L.hipGraphDestroy(graph) == 0
    print("[gpu] eager backward after it", flush=True)
    C.check(L.mt_batch_backward(b.h, *tabs, 0, b._s()))
    torch.cuda.synchronize()
    assert all(equal_outs(x, r) for x, r in zip(g, ref_g))
