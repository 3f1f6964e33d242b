"""GPU parity of large batches in ordinary host memory, whose columns several threads copy: sizes on both sides of the line, one after
the other on one context, and from two threads at once."""
import threading

import numpy as np
import pytest

from oracle import ccld_oracle as orc
from paper_2605_04478_amd import ccld, tracegen as tg
from tests.helpers import T0
from tests.test_gpu_window import FAR, compare

pytestmark = pytest.mark.gpu

LINE = (32 << 20) // 41              # records of 41 bytes


def _cols(n, seed):
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    te = T0 + i // 256 * 10**6 + rng.integers(0, 1000, n)
    te[rng.random(n) < 0.001] += 10**8
    return {"rank": (i % 256).astype(np.uint32), "comm": (i % 256 // 64).astype(np.uint32), "seq": (i // 256).astype(np.uint64),
            "op": np.ones(n, np.uint8), "bytes": np.full(n, 4096, np.uint64), "t_enter": te, "t_exit": te + 5 * 10**8}


TOPO = [list(range(i, i + 64)) for i in range(0, 256, 64)]


def _run(sizes, seed, out):
    topo = tg.make_topology(256, TOPO)
    an = ccld.Analyzer(topo, max_window_records=LINE + 4096)
    for k, n in enumerate(sizes):
        an.reset_window()
        cols = _cols(n, seed + k)
        an.ingest({k: v.copy() for k, v in cols.items()})        # gone once the call returns
        out.append((cols, an.analyze_window(FAR, n_records=n), an.rank_blame()))
    an.close()


@pytest.fixture(scope="module", autouse=True)
def helping_threads():
    """a context that has handed over so much that threads help with large batches, its own and those of the contexts below"""
    an = ccld.Analyzer(tg.make_topology(256, TOPO), max_window_records=LINE + 4096)
    cols = _cols(LINE + 1, 99)
    for _ in range(34):
        an.reset_window()
        an.ingest(cols)
    yield an, cols
    an.close()


def _check(out):
    o = orc.Oracle(tg.make_topology(256, TOPO))
    for cols, g, (blame, order) in out:
        compare(g, o.analyze_window(cols, FAR), blame, order, per_record=False, what=cols["rank"].size)


def test_batches_on_both_sides_of_the_line():
    out = []
    _run([LINE + 1, 500, LINE, LINE + 4096], 1, out)
    assert len(out) == 4
    _check(out)


def test_batches_before_and_after_the_threads_help(helping_threads):
    an, cols = helping_threads
    for _ in range(2):
        an.reset_window()
        an.ingest({k: v.copy() for k, v in cols.items()})
        _check([(cols, an.analyze_window(FAR, n_records=LINE + 1), an.rank_blame())])


def test_two_contexts_in_two_threads():
    outs = [[], []]
    threads = [threading.Thread(target=_run, args=([LINE + 77, LINE + 300], 10 * (t + 1), outs[t])) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for out in outs:
        assert len(out) == 2
        _check(out)
