"""Clocks of up to 64 GPUs travel with a launch, those of more are read from
a table in device memory: records, markers and dispatch times on either side
of that and at the largest number of GPUs, with clocks that all differ."""
import dataclasses

import numpy as np
import pytest

import oracle
import tracegen as tg
from test_gpu_launch import split_both
from test_gpu_parity import (assert_parity, ch, natural_order,  # noqa: F401
                             run_gpu, say)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["any", "profiler"])
@pytest.mark.parametrize("gpus", [63, 64, 65, 128, 256])
def test_clocks(ch, gpus, order):
    say("clocks of", gpus, "GPUs,", order)
    tr = tg.make_micro(gpus, n_gpus=gpus, n_kernels=6000, n_streams=2, depth=3,
                       span=40_000, n_counters=2, anchors=6)
    if order == "profiler":
        tr = natural_order(tr)
    ref = oracle.run(tr)
    assert len(np.unique(ref["c"])) > gpus // 2
    assert_parity(run_gpu(ch, tr), ref, name=f"{gpus} GPUs {order}")


@pytest.mark.parametrize("gpus", [64, 65, 256])
def test_launch_split(ch, gpus):
    import torch
    say("launch split of", gpus, "GPUs")
    tr = tg.make_micro(gpus, n_gpus=gpus, n_kernels=5000, n_streams=2, depth=2,
                       span=30_000, anchors=6)
    tl = tg.make_launch(tr, 5, max_lead=300)
    (gp, gc), (rp, rc), st, r = split_both(ch, tr, tl)
    assert np.array_equal(gp, rp) and np.array_equal(gc, rc)
    assert st == r["status"]
    pipe = ch.Pipeline(ch.DeviceTrace(tr, "cuda"))
    pipe.step()
    p, c = pipe.launch_split_noalloc(torch.from_numpy(tl).cuda())
    assert np.array_equal(p.cpu().numpy(), rp)
    assert np.array_equal(c.cpu().numpy(), rc)


def test_a_record_past_the_table(ch):
    """A GPU id above the number of GPUs: reported, on either side."""
    for gpus in (64, 65):
        say("GPU id out of range beside", gpus)
        tr = tg.make_micro(9, n_gpus=gpus, n_kernels=2000, n_streams=2,
                           depth=2, span=20_000, anchors=4)
        g = tr.gpu.copy()
        g[17] = gpus
        got = run_gpu(ch, dataclasses.replace(tr, gpu=g))
        assert got["status"] & 1
