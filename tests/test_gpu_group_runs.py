"""Rows of groups that are not one run of records (lost markers, markers in
any numbering, selections): the tiles' election against the oracle, bit for
bit, around the 512-record tile and over every record order."""
import dataclasses

import numpy as np
import pytest

import oracle
import tracegen as tg
from test_gpu_parity import assert_parity, ch, natural_order, run_gpu, say

pytestmark = pytest.mark.gpu


def opened(tr):
    """Markers numbered in the order they open."""
    o = np.lexsort((tr.m_level, tr.m_start, tr.m_gpu))
    return dataclasses.replace(
        tr, m_gpu=tr.m_gpu[o], m_level=tr.m_level[o], m_start=tr.m_start[o],
        m_end=tr.m_end[o], m_label=tr.m_label[o])


def cut(tr, n):
    """The first n records."""
    r = {k: getattr(tr, k)[:n] for k in ("gpu", "stream", "start", "end",
                                         "cls", "op_id")}
    ctr = None if tr.counters is None else tr.counters[:, :n].copy()
    return dataclasses.replace(tr, counters=ctr, **r)


def merged(tr):
    p = np.argsort(tr.start, kind="stable")
    ctr = None if tr.counters is None else tr.counters[:, p]
    return dataclasses.replace(
        tr, counters=ctr, **{k: getattr(tr, k)[p] for k in (
            "gpu", "stream", "start", "end", "cls", "op_id")})


def lost_markers(seed, iters=1, order="profiler", numbered="opened"):
    """Two compute and two communication streams, markers of depth 3 to 6,
    three in a hundred of them lost on top of the generator's."""
    tr = natural_order(tg.make_config(4, iters=iters, seed=seed))
    keep = np.random.default_rng(seed).random(tr.n_markers) >= 0.03
    tr = dataclasses.replace(
        tr, **{k: getattr(tr, k)[keep] for k in (
            "m_gpu", "m_level", "m_start", "m_end", "m_label")})
    if numbered == "opened":
        tr = opened(tr)
    return merged(tr) if order == "merged" else tr


@pytest.mark.parametrize("n", [1, 511, 512, 513, 1024, 3073, 24576])
@pytest.mark.parametrize("order,numbered", [
    ("profiler", "opened"), ("profiler", "any"), ("merged", "opened")])
def test_lost_markers(ch, n, order, numbered):
    tr = cut(lost_markers(11, order=order, numbered=numbered), n)
    say("lost markers", n, order, numbered)
    ref = oracle.run(tr)
    assert_parity(run_gpu(ch, tr), ref, name=f"lost {n} {order} {numbered}")


@pytest.mark.parametrize("level", [0, 2, 4, 5, 100])
def test_lost_markers_single_level(ch, level):
    tr = lost_markers(12)
    say("lost markers, level", level)
    assert_parity(run_gpu(ch, tr, level=level), oracle.run(tr, level=level),
                  name=f"lost, level {level}")


SELECT = [dict(iters=(1, 2)), dict(iters=(7, 9)), dict(gpus=[1, 5]),
          dict(classes=[5, 6]), dict(gpus=[0, 7], classes=[0, 6],
                                     iters=(0, 1))]


@pytest.mark.parametrize("sel", range(len(SELECT)))
@pytest.mark.parametrize("kind", ["runs", "lost", "merged"])
@pytest.mark.parametrize("level", [255, 2, 100])
def test_selections(ch, sel, kind, level):
    """Iterations, GPUs and classes left out: one compute stream and tiling
    markers, lost markers, and ranks merged by time."""
    if kind == "lost":
        tr = lost_markers(13, iters=3)
    else:
        tr = tg.make_config(1, iters=3, seed=14)
        tr = merged(tr) if kind == "merged" else tr
    say("selection", SELECT[sel], kind, level)
    ref = oracle.run(tr, level=level, filt=oracle.make_filter(**SELECT[sel]))
    got = run_gpu(ch, tr, level=level, filt=ch.make_filter(**SELECT[sel]))
    assert_parity(got, ref, name=f"selection {sel} {kind} {level}")


def test_capacity(ch):
    """Fewer row slots than rows: the offsets hold the needed counts and the
    flag is set."""
    import torch
    tr = lost_markers(15)
    pipe = ch.Pipeline(ch.DeviceTrace(tr, "cuda"))
    pipe.step()
    torch.cuda.synchronize()
    want = pipe.rows.level_offset.cpu().numpy().copy()
    assert want[-1] > 1000
    pipe.rows = ch.RowsBuffer(1000, tr.depth, tr.n_counters, "cuda")
    pipe._scr["aggregate"] = torch.empty(
        pipe._scr["aggregate"].numel(), dtype=torch.uint8, device="cuda")
    pipe.status.zero_()
    pipe.aggregate()
    torch.cuda.synchronize()
    assert np.array_equal(pipe.rows.level_offset.cpu().numpy(), want)
    assert pipe.status.item() & ch.ST_ROWS_OVERFLOW


@pytest.mark.parametrize("depth,filt", [(6, None), (8, dict(
    iters=(3, 40), gpus=[0, 1, 2, 5, 6], classes=[0, 1, 2, 5, 6, 7]))])
def test_records_in_no_order(ch, depth, filt):
    """Enough shuffled records for the pass through rows, paths of six and
    eight levels, the latter with a selection."""
    tr = tg.make_config(4, iters=43, seed=17)
    assert tr.n >= 1 << 20
    tr = dataclasses.replace(tr, depth=depth)
    say("no order", tr.n, depth, filt)
    of = None if filt is None else oracle.make_filter(**filt)
    cf = None if filt is None else ch.make_filter(**filt)
    assert_parity(run_gpu(ch, tr, filt=cf), oracle.run(tr, filt=of),
                  name=f"no order, depth {depth}")


@pytest.mark.parametrize("counters,level", [(0, 255), (1, 255), (3, 1),
                                            (4, 100), (5, 255), (16, 2)])
def test_no_order_column_groups(ch, counters, level):
    """The same pass takes four columns at a time: groups that are whole, that
    are cut short and that are left out, at all levels and at one."""
    from test_gpu_periodic_gaps import periodic
    tr = periodic((1 << 19) + 77, (256, 64, 4), (0,), 3, n_counters=counters,
                  gpus=2)
    p = np.random.default_rng(counters).permutation(tr.n)
    tr = dataclasses.replace(
        tr, counters=None if tr.counters is None else tr.counters[:, p],
        **{k: getattr(tr, k)[p] for k in ("gpu", "stream", "start", "end",
                                          "cls", "op_id")})
    assert tr.n >= 1 << 20
    say("no order,", counters, "counters, level", level)
    assert_parity(run_gpu(ch, tr, level=level), oracle.run(tr, level=level),
                  name=f"no order, {counters} counters, level {level}")
