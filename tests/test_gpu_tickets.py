"""The calls around the number at which the tags of the reports start over: each still answers for its own window."""
import pytest

from tests.helpers import ring_topology, rounds_with_durations, toy_cols
from tests.test_gpu_window import FAR

pytestmark = pytest.mark.gpu


def test_reports_where_the_tags_start_over():
    from paper_2605_04478_amd import ccld
    rows = [rounds_with_durations([[100, 200, 300, 400]] * k) for k in (3, 5)]
    an = ccld.Analyzer(ring_topology(4), max_window_records=64)
    windows = [(an.to_device(toy_cols(rows[0])), "OK", 3), (an.to_device(toy_cols(rows[1])), "OK", 5),
               (an.to_device(toy_cols(rows[1] + rows[1][:1])), "E_DUPLICATE_KEY", 0)]
    buffers = an.alloc_window_result(64)
    blame = None

    def analyze(k):
        cols, status, n_seg = windows[k % 3]
        an.reset_window()
        an.ingest(cols)
        res = an.analyze_window(FAR, buffers=buffers)
        assert (res.status, res.n_seg) == (status, n_seg), k

    analyze(0)                                  # the first ticket
    for _ in range(65_536 - 8):                 # one ticket each
        blame = an.rank_blame(to_host=False, buffers=blame and (blame[0].view(-1), blame[1]))
    for k in range(1, 16):
        analyze(k)
    an.close()
