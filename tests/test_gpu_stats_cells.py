"""Per-GPU overlap CDFs of chopper_op_stats by the length of a CDF group: one
wave selects it up to 128 slots (up to 1,024 where more than 512 groups are
longer), one block up to 32,768 instances, parts of 8,192 above that.  Lengths
at the edges of all of them, GPUs that follow each other and GPUs mixed row by
row, ratios with many ties, bit for bit against the CPU oracle."""
import numpy as np
import pytest

import oracle
import tracegen as tg
from test_gpu_stats import ch, check, say  # noqa: F401

pytestmark = pytest.mark.gpu


def stats_of_rows(ch, gpu, phase, op, n_gpus, n_phases, n_ops, seed, ties):
    """Rows of one level pair (phase, operation) given per row."""
    import torch
    n = len(gpu)
    rng = np.random.default_rng(seed)
    tr = tg.make_micro(3, n_gpus=n_gpus, n_kernels=300, depth=2, span=3000,
                       n_counters=16)
    i = np.arange(128)
    tr.m_gpu, tr.m_level = np.zeros(128, np.uint8), np.zeros(128, np.uint8)
    tr.m_start, tr.m_end = i * 10, i * 10 + 5
    tr.m_label = i.astype(tr.m_label.dtype)
    dur = rng.integers(1, 50_000, n) * 8
    kinds = rng.integers(0, 5, n)
    ovl = np.where(kinds == 0, 0, np.where(kinds == 1, dur, np.where(
        kinds == 2, dur // 8 * rng.integers(1, 8, n),
        rng.integers(0, 1 << 62, n) % (dur + 1))))
    if ties:
        ovl = np.where(kinds < 4, dur // 2, 0)
    rows = dict(
        level_offset=np.array([0, 0, n, n, n], np.int64), n_rows=n,
        path=np.stack([phase, op]).astype(np.uint32),
        gpu=gpu.astype(np.uint8), kind=np.zeros(n, np.uint8),
        n=np.ones(n, np.uint64), dur=dur.astype(np.uint64),
        gap=rng.integers(0, 3000, n).astype(np.uint64),
        ovl=ovl.astype(np.uint64), tmin=np.zeros(n, np.int64),
        tmax=dur.astype(np.int64), first=np.arange(n, dtype=np.uint32),
        ctr=rng.integers(0, 1 << 40, (16, n)).astype(np.uint64))
    buf = ch.RowsBuffer(n, 2, 16, "cuda")
    for k, v in rows.items():
        if k != "n_rows":
            t = getattr(buf, k)
            t.copy_(torch.from_numpy(v.view(
                {1: np.uint8, 4: np.int32, 8: np.int64}[v.itemsize])))
    pipe = ch.Pipeline(ch.DeviceTrace(tr, "cuda"))
    pipe.rows = buf
    pipe.status.zero_()
    spec = dict(n_phases=n_phases, n_ops=n_ops, phase_level=0, op_level=1)
    for _ in range(2):                      # (the second on used scratch)
        out, cnt, gout, gcnt = pipe.op_stats(per_gpu=True, **spec)
    got = (out.cpu().numpy(), cnt.cpu().numpy(), 0, gout.cpu().numpy(),
           gcnt.cpu().numpy())
    return got, oracle.op_stats(rows, tr.m_label, 2, n_gpus=n_gpus,
                                per_gpu=True, **spec)


LENGTHS = [1, 2, 3, 63, 64, 65, 127, 128, 129, 511, 512, 513, 540, 960, 1023,
           1024, 1025, 8193]


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("lengths", [
    LENGTHS, [32_767, 32_768, 32_769, 34_500, 34_600, 40],
    [150_001], [69_000, 5, 36_001, 2_000]])
def test_lengths(ch, lengths, mixed, ties):
    """Rows of an operation each on two of three GPUs."""
    say("op stats: CDF groups of", lengths, "mixed" if mixed else "in turn",
        "ties" if ties else "")
    rng = np.random.default_rng(len(lengths))
    op = np.concatenate([np.repeat(np.arange(len(lengths)), lengths)] * 2)
    gpu = np.repeat([0, 2], len(op) // 2)
    o = rng.permutation(len(op))
    if not mixed:
        o = o[np.argsort(gpu[o], kind="stable")]
    got, ref = stats_of_rows(ch, gpu[o], np.zeros(len(op), np.int64), op[o], 3,
                             1, len(lengths), 11, ties)
    check(got, ref, f"lengths {lengths}")
    assert (got[4].reshape(-1, 3)[:, 1] == 0).all()


@pytest.mark.parametrize("gpus,rows", [(1, 3_000), (8, 200_000),
                                       (256, 120_000)])
def test_most_groups(ch, gpus, rows):
    """16 phases of 128 operations on up to 256 GPUs: every way of listing,
    most CDF groups small or empty."""
    say("op stats: 2,048 groups on", gpus, "GPUs")
    rng = np.random.default_rng(gpus)
    gpu = np.sort(rng.integers(0, gpus, rows))
    # a few operations hold most of the rows
    op = np.minimum(rng.geometric(0.08, rows) - 1, 127)
    got, ref = stats_of_rows(ch, gpu, rng.integers(0, 16, rows), op, gpus, 16,
                             128, 5, False)
    check(got, ref, f"{gpus} GPUs")
    assert (got[4] > 0).sum() > 500 and (got[4] == 0).any()


def test_gpu_boundary_in_one_block(ch):
    """GPUs that end inside blocks of 4,096 rows, one group: those blocks add
    their instances by GPU."""
    say("op stats: GPUs of 700 rows each, one group")
    gpu = np.repeat(np.arange(30), 700)
    z = np.zeros(len(gpu), np.int64)
    got, ref = stats_of_rows(ch, gpu, z, z, 29, 1, 1, 2, False)
    check(got, ref, "one group, 30 GPUs of which 29 count")


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("groups,length", [(512, 140), (513, 140), (600, 129),
                                           (600, 513), (640, 1023),
                                           (640, 1024), (640, 1025)])
def test_many_middle_groups(ch, groups, length, mixed):
    """About 512 groups longer than 128, which go to waves above that."""
    say("op stats:", groups, "CDF groups of", length,
        "mixed" if mixed else "in turn")
    # a group a phase, operation and GPU
    cell = np.repeat(np.arange(groups), length)
    gpu, rest = cell % 8, cell // 8
    o = np.random.default_rng(groups + length).permutation(len(cell))
    if not mixed:
        o = o[np.argsort(gpu[o], kind="stable")]
    got, ref = stats_of_rows(ch, gpu[o], rest[o] % 3, rest[o] // 3, 8, 3, 64,
                             17, length % 2 == 0)
    check(got, ref, f"{groups} of {length}")
    assert (got[4] == length).sum() == groups
