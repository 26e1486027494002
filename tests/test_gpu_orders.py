"""The two record orders for input in no order: spans that fit one sort by
time for both and spans that do not, more than 256 (gpu, stream) pairs, equal
times, and ranks merged by time (element by element against the oracle)."""
import dataclasses

import numpy as np
import pytest

import oracle
import tracegen as tg
from test_gpu_parity import assert_parity, ch, run_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [1, 8, 16, 40, 47, 49, 58])
@pytest.mark.parametrize("n", [2, 2047, 2049, 6000])
def test_time_spans(ch, bits, n):
    say("orders: times over", bits, "bits,", n, "records")
    rng = np.random.default_rng(bits * 10007 + n)
    tr = tg.make_micro(bits + n, n_gpus=3, n_kernels=n, n_streams=4, depth=2)
    start = rng.integers(0, 1 << bits, n).astype(np.int64)
    start[:2] = 0, (1 << bits) - 1
    end = start + rng.integers(0, 1 << min(bits, 20), n)
    tr = dataclasses.replace(tr, start=start, end=end)
    assert_parity(run_gpu(ch, tr), oracle.run(tr), name=f"{bits} bits, {n}")


@pytest.mark.parametrize("streams", [80, 100])
def test_many_streams(ch, streams):
    """240 pairs (one sort by time) and 300 (one sort per order)."""
    say("orders:", streams, "streams on three GPUs")
    tr = tg.make_micro(streams, n_gpus=3, n_kernels=9000, n_streams=streams,
                       depth=2, nested=False, span=1 << 22)
    assert_parity(run_gpu(ch, tr), oracle.run(tr), name=f"{streams} streams")


def test_merged_then_one_late(ch):
    """Ranks merged by time, and the same with one record out of place."""
    tr = tg.make_config(1, iters=1, seed=21)
    p = np.argsort(tr.start, kind="stable")
    for swap in (False, True):
        say("orders: merged", "with one late" if swap else "")
        if swap:
            p[[100, -100]] = p[[-100, 100]]
        part = {k: getattr(tr, k)[p] for k in (
            "gpu", "stream", "start", "end", "cls", "op_id")}
        m = dataclasses.replace(tr, **part)
        assert_parity(run_gpu(ch, m), oracle.run(m), name=f"merged {swap}")
