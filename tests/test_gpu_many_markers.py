"""More markers than records: up to 2^20 of them the overlap queries of fewer
records than that share a launch, from there on they have their own."""
import pytest

import oracle
from test_gpu_parity import assert_parity, ch, run_gpu, say  # noqa: F401
from test_gpu_periodic_gaps import periodic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("records", [131_071, 131_072, 131_073])
def test_eight_markers_a_record(ch, records):
    """Eight levels of one marker a record: 2^20 - 8, 2^20 and 2^20 + 8."""
    tr = periodic(records, (1,) * 8, (), comm_every=7, n_counters=0)
    say("markers", tr.n_markers, "records", tr.n)
    assert tr.n_markers == 8 * records
    assert_parity(run_gpu(ch, tr), oracle.run(tr), name=f"{records} records")
