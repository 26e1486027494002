"""The passes of a join in one launch a kernel and pass by pass: (gpu, stream)
pairs on both sides of what one class table holds, passes of unequal lengths
around the tiles of the partition, entries without an iteration between runs
and a pass whose labels are not one run each (element by element against the
oracle)."""
import numpy as np
import pytest

import oracle
import tracegen as tg
from test_gpu_join import NONE, ch, check, join_both, say

pytestmark = pytest.mark.gpu


def with_labels(tr):
    r0 = oracle.run(tr)
    idx = r0["idx"].reshape(-1, tr.n)[0]
    lab = np.full(tr.n, NONE, np.uint32)
    lab[idx != NONE] = tr.m_label[idx[idx != NONE]]
    return lab


@pytest.mark.parametrize("streams", [11, 12, 60])
@pytest.mark.parametrize("variant", [0, 1, 2])
def test_pairs_and_lengths(ch, streams, variant):
    """33 pairs (one table for seven passes), 36 and 180 (pass by pass)."""
    say("join passes:", streams, "streams on three GPUs, variant", variant)
    tr = tg.make_micro(streams + variant, n_gpus=3, n_kernels=7000,
                       n_streams=streams, depth=2, n_counters=16,
                       nested=False, span=1 << 20)
    passes = tg.make_counter_passes(tr, with_labels(tr), variant,
                                    drop_frac=0.02 * variant,
                                    mismatch_frac=0.01 * variant)
    for q, m in zip(passes, [None, 2047, 2048, 2049, 1, 255, 257]):
        if variant and m:
            for k in ("gpu", "stream", "cls", "lab"):
                q[k] = q[k][:m].copy()
            q["values"] = np.ascontiguousarray(q["values"][:, :m])
    if variant == 1:                 # no iteration at every seventh entry
        passes[0]["lab"][::7] = NONE
    if variant == 2:                 # one pass's labels in no order
        passes[0]["lab"] = np.random.default_rng(streams).permutation(
            passes[0]["lab"])
    got, ref, _ = join_both(ch, tr, passes)
    check(got, ref, f"{streams} streams, variant {variant}")
