"""mt_batch_build on another stream than a batch call still in flight: the
build waits for it before it overwrites the tables that its kernels read."""

import ctypes

import pytest
import torch

import synth
from tests.test_gpu_batch import equal_outs, make_ifaces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_graph", [0, 1])
def test_build_beside_a_running_forward(use_graph):
    from paper_2202_03933_amd import MortarBatch
    from paper_2202_03933_amd import _capi as C
    from paper_2202_03933_amd.batch import _ptr_table
    ifaces = make_ifaces(synth.batched_instances(n_inst=4, max_side=32))
    ref = [tuple(t.clone() for t in it.integrate()) for it in ifaces]
    b = MortarBatch(ifaces)
    outs = b.alloc_outputs()
    tabs = [_ptr_table([o[k] for o in outs]) for k in range(3)]
    other = torch.cuda.Stream()
    long = torch.empty(1 << 27, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    run = lambda: C.check(C.lib().mt_batch_forward(b.h, *tabs, use_graph, b._s()))
    run()  # uploads the output pointers: the next call waits for nothing
    torch.cuda.synchronize()
    for o in outs:
        for t in o:
            t.fill_(float("nan"))
    torch.cuda.synchronize()
    print(f"[gpu] batch build beside a queued forward, graph={use_graph}", flush=True)
    with torch.cuda.stream(b.stream):
        for _ in range(100):  # about 20 ms ahead of the forward
            long.zero_()
    run()
    t = C.mt_batch_tuning()
    C.check(C.lib().mt_batch_build(b.h, ctypes.byref(t), ctypes.c_void_p(b._ws_ptr), b._ws_bytes,
                                   ctypes.c_void_p(other.cuda_stream)))
    torch.cuda.synchronize()
    assert all(equal_outs(o, r) for o, r in zip(outs, ref))
    run()  # and with the tables of the new build
    torch.cuda.synchronize()
    assert all(equal_outs(o, r) for o, r in zip(outs, ref))
