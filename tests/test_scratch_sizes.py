"""Scratch that chopper_aggregate asks for (a size query does no GPU work): a
path for records in no order must not make every caller pay for it."""
import ctypes

import pytest

import paper_2512_08242_amd as ch

b = ch.binding
FAKE = ctypes.c_void_p(0x1000)


def aggregate_bytes(n, markers, depth, counters, cap, level=255):
    def fill(s, **kw):
        for f, t in s._fields_:
            if t is b.P:
                setattr(s, f, FAKE)
        for k, v in kw.items():
            setattr(s, k, v)
        return s
    rec = fill(b.Records(), n=n, n_gpus=8, n_counters=counters)
    mk = fill(b.Markers(), n=markers, depth=depth) if depth else None
    rows = fill(b.Rows(), cap=cap)
    sz = ctypes.c_size_t()
    assert ch.lib.chopper_aggregate(
        ctypes.byref(rec), FAKE, FAKE, FAKE, FAKE, depth, FAKE, FAKE,
        ctypes.byref(mk) if mk else None, level, None, ctypes.byref(rows),
        None, ctypes.byref(sz), None, None, None) == 0
    return sz.value


@pytest.mark.parametrize("level", [255, 0, 100])
@pytest.mark.parametrize("depth", [0, 1, 4, 6, 8])
def test_no_step_at_any_size(depth, level):
    """Bytes a record stay the same over the sizes, whichever passes a size
    has, and do not grow with the counters."""
    if level == 0 and depth == 0:
        pytest.skip("no marker level")
    per = []
    for n in ((1 << 20) - 512, 1 << 20, 1 << 22, 1 << 25, (1 << 29) - 512):
        q = aggregate_bytes(n, n // 4, depth, 16, n // 3, level)
        assert q == aggregate_bytes(n, n // 4, depth, 0, n // 3, level)
        per.append(q / n)
    # (tables of fixed size: a few bytes a record at 2^20)
    assert max(per) < min(per) + 10


def test_headline_sizes():
    """19.66M records with 16 counters and 7.2M row slots at depth 4; the
    largest call of depth 4."""
    assert aggregate_bytes(19_660_800, 6_387_200, 4, 16, 7_200_000) < 2.36e9
    n = (1 << 29) - 1
    assert aggregate_bytes(n, 1 << 28, 4, 16, 1 << 28) < 64.6e9
