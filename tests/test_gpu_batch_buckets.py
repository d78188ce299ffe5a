"""Pairs per work item of a batch: the smallest, ones that are no whole tiles
of 64 pairs, and the largest that the tuning's field holds (one item per
interface) give the values of the default."""

import pytest
import torch

import synth
from tests.test_gpu_batch import equal_outs, make_ifaces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bucket", [1, 63, 65, 1000, 2**31 - 65, 2**31 - 64, 2**31 - 63, 2**31 - 1])
def test_bucket(bucket):
    from paper_2202_03933_amd import MortarBatch
    ifaces = make_ifaces(synth.batched_instances(n_inst=4, max_side=32))
    ref = [tuple(t.clone() for t in it.integrate()) for it in ifaces]
    print(f"[gpu] batch with buckets of {bucket} pairs", flush=True)
    outs = MortarBatch(ifaces, tuning={"bucket": bucket}).forward()
    torch.cuda.synchronize()
    assert all(equal_outs(o, r) for o, r in zip(outs, ref))
