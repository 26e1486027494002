"""Rows of groups of several runs whose outer markers come and go with a
period that lines up with the 512-record tiles (iterations of a fixed number
of kernels, every second marker of an outer level lost): nearly every tile
then starts with a group that came before, at more than one level, so the
pieces that are added to the rows afterwards are as many as they can get."""
import numpy as np
import pytest

import oracle
import tracegen as tg
from test_gpu_group_runs import merged
from test_gpu_parity import assert_parity, ch, run_gpu, say

pytestmark = pytest.mark.gpu

STEP = 100


def periodic(n, spans, lost, comm_every=0, n_counters=2, gpus=1, seed=5):
    """n records on each of `gpus` GPUs, one every 100 ns; level l's markers
    cover spans[l] records each (a pair: on average so many to so many
    markers), every second one of the levels in `lost`,
    the first one on, is missing.  comm_every: every so many records a communication kernel."""
    rng = np.random.default_rng(seed)
    i = np.arange(n, dtype=np.int64)
    start = 1_000_000 + i * STEP
    cls = np.where(comm_every > 0 and i % max(comm_every, 1) == 1, 5,
                   i % 5).astype(np.uint8)
    stream = (cls == 5).astype(np.uint8)
    mk = [[], [], [], []]                     # level, start, end, label
    for l, span in enumerate(spans):
        num, den = span if isinstance(span, tuple) else (span, 1)
        j = np.arange(-(-n * den // num))
        if l in lost:
            j = j[1::2]
        mk[0].append(np.full(len(j), l, np.uint8))
        mk[1].append(1_000_000 + j * num // den * STEP)
        mk[2].append(1_000_000 + np.minimum((j + 1) * num // den, n) * STEP)
        mk[3].append(j.astype(np.uint32) % 97)
    lev, ms, me, lab = (np.concatenate(x) for x in mk)
    o = np.lexsort((lev, ms))
    m = len(o)
    rep = lambda x: np.tile(x, gpus)
    return tg.Trace(
        n_gpus=gpus, depth=len(spans),
        gpu=np.repeat(np.arange(gpus, dtype=np.uint8), n), stream=rep(stream),
        start=rep(start), end=rep(start) + rng.integers(1, 90, n * gpus),
        cls=rep(cls), op_id=np.zeros(n * gpus, np.uint32),
        counters=rng.integers(0, 1 << 40, (n_counters, n * gpus)).astype(
            np.uint64) if n_counters else None,
        m_gpu=np.repeat(np.arange(gpus, dtype=np.uint8), m),
        m_level=rep(lev[o]), m_start=rep(ms[o]).astype(np.int64),
        m_end=rep(me[o]).astype(np.int64), m_label=rep(lab[o]),
        a_gpu=np.zeros(0, np.uint8), a_local=np.zeros(0, np.int64),
        a_ref=np.zeros(0, np.int64))


# records, marker spans, levels with every second marker lost, spacing of
# communication kernels
GAPS = {
    # 256 records inside and 256 outside the two outer markers
    "depth 4": (245_760, (256, 256, 16, 2), (0, 1), 9),
    "depth 3": (524_288, (128, 32, 4), (0,), 9),
    # 480 rows to an iteration of 512 records, one kind only
    "480 rows": (524_288, (512, (16, 15), 1), (0,), 0),
    "depth 5": (245_760, (256, 256, 64, 16, 2), (0, 1, 2), 9),
    "depth 7": (262_144, (512, 256, 128, 64, 32, 8, 2), (0, 1, 3), 5),
    "depth 8": (131_072, (512, 512, 256, 128, 64, 32, 4, 1), (0, 2, 4), 5),
    "outer only": (262_144, (512,), (0,), 2),
    "depth 2": (262_144, (256, 64), (0,), 3),
}


@pytest.mark.parametrize("order", ["profiler", "merged"])
@pytest.mark.parametrize("which", GAPS)
def test_periodic_gaps(ch, which, order):
    n, spans, lost, comm = GAPS[which]
    tr = periodic(n, spans, lost, comm)
    if order == "merged":
        # a second GPU, so that the records are not grouped by GPU
        tr = merged(periodic(n // 2, spans, lost, comm, gpus=2))
    say("periodic gaps", which, order, tr.n, tr.n_markers)
    assert_parity(run_gpu(ch, tr), oracle.run(tr), name=f"{which} {order}")


@pytest.mark.parametrize("which", ["depth 4", "depth 3"])
def test_periodic_gaps_selected(ch, which):
    n, spans, lost, comm = GAPS[which]
    tr = periodic(n, spans, lost, comm)
    say("periodic gaps, selection", which)
    filt = dict(classes=[0, 1, 2, 4, 5])
    assert_parity(run_gpu(ch, tr, filt=ch.make_filter(**filt)),
                  oracle.run(tr, filt=oracle.make_filter(**filt)),
                  name=f"{which} selected")
