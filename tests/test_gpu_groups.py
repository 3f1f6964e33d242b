"""GPU parity of the detection groups where their kernels can go wrong: more groups in one communicator than one
baseline walk takes, baselines that end by count and by time inside a window, and more communicators than the group
table's wavefronts sum by themselves."""
import numpy as np
import pytest

from oracle import ccld_oracle as orc
from paper_2605_04478_amd import tracegen as tg
from tests.helpers import T0, ring_topology, toy_cols
from tests.test_gpu_window import FAR, compare

pytestmark = pytest.mark.gpu


def _windows(topo, windows, **params):
    from paper_2605_04478_amd import ccld
    n = max(len(w) for w in windows)
    an = ccld.Analyzer(topo, max_window_records=n, **params)
    o = orc.Oracle(topo, params)
    ref = None
    for i, rows in enumerate(windows):
        cols = toy_cols(rows)
        p = np.random.default_rng(i).permutation(len(rows))
        cols = {k: v[p] for k, v in cols.items()}
        an.reset_window()
        an.ingest(an.to_device(cols))
        g, ref = an.analyze_window(FAR, n_records=n, per_record=True), o.analyze_window(cols, FAR)
        compare(g, ref, *an.rank_blame(), what=f"window{i}")
    an.close()
    return ref


@pytest.mark.parametrize("groups", [63, 64, 65, 200])
@pytest.mark.parametrize("rounds,tbase_rounds", [(1, 3), (4, 3), (9, 100)])
def test_many_groups_in_one_communicator(groups, rounds, tbase_rounds):
    topo = ring_topology(3, comms=[[0, 1, 2], [2, 1]])
    rng = np.random.default_rng(groups + rounds)
    windows, seq = [], 0
    for w in range(3):
        rows = []
        for j in range(rounds):
            for g in rng.permutation(groups):
                t = T0 + (w * rounds + j) * 1_000_000_000 + int(g) * 1000
                for r in range(3):
                    d = 1000 + int(rng.integers(0, 9000))
                    rows.append((r, 0, seq, int(g) % 16, 1 << (4 + int(g) // 16), t, t + d))
                seq += 1
            rows += [(r, 1, w * rounds + j, 0, 64, T0 + j, T0 + j + 7 + r) for r in (1, 2)]
        windows.append(rows)
    ref = _windows(topo, windows, tbase_rounds=tbase_rounds, tbase_init_ns=2000, tbase_warmup_ns=6_000_000_000)
    assert len(ref.group["comm"]) == groups + 1


def test_more_communicators_than_one_wavefront_sums():
    n = 8200
    topo = tg.make_topology(n, [[i, (i + 1) % n] for i in range(n)])
    rows = [(r, c, s, (c + s) % 3, 1 << 20, T0 + s * 1000, T0 + s * 1000 + 100 + r % 7)
            for c in range(0, n, 3) for s in range(2) for r in (c, (c + 1) % n)]
    ref = _windows(topo, [rows], tbase_init_ns=50)
    assert len(ref.group["comm"]) == 2 * len(range(0, n, 3))


@pytest.mark.parametrize("tbase_rounds,warmup_rounds", [(1, 10**6), (4095, 10**6), (4096, 10**6), (4097, 10**6), (100, 4096), (10**6, 4095),
                                                        (5000, 5000), (10**6, 10**6)])
def test_baselines_that_end_at_the_edges_of_a_walk(tbase_rounds, warmup_rounds):
    """A communicator of 9,000 rounds per window: baselines that end by their count or by the warm-up span in the first
    step of the walk over its rows, at its edges, later or not at all, a group of its own every 700 rounds, and one that
    only the second window has."""
    topo = ring_topology(2)
    SPACING = 1000
    windows = []
    for w in range(3):
        rows, rng = [], np.random.default_rng(w)
        for j in range(w * 9000, (w + 1) * 9000):
            t, op = T0 + j * SPACING, 3 if j % 700 == 699 else 5 if 9000 <= j < 18000 and j % 50 == 7 else 0
            rows += [(r, 0, j, op, 1 << 20, t, t + 100 + int(d)) for r, d in enumerate(rng.integers(0, 900, 2))]
        windows.append(rows)
    ref = _windows(topo, windows, tbase_rounds=tbase_rounds, tbase_init_ns=300, tbase_warmup_ns=warmup_rounds * SPACING)
    assert len(ref.group["comm"]) == 2


@pytest.mark.parametrize("rounds", [1, 511, 512, 513, 2047, 2048, 2049, 4095, 4096, 4097])
def test_rows_at_the_edges_of_a_step(rounds):
    """the slowest round of a group in the first, a middle or the last row of its communicator; equal ones, of which the first counts"""
    topo = ring_topology(3, comms=[[0, 1], [1, 2, 0], [2, 1]])
    rng = np.random.default_rng(rounds)
    windows = []
    for w, slow in enumerate(([0], [rounds // 2, rounds - 1], [rounds - 1])):
        rows = []
        for c in range(3):
            for j in range(rounds):
                t = T0 + (w * rounds + j) * 1_000_000
                for r in topo.members_of(c):
                    rows.append((int(r), c, w * rounds + j, j % 2, 64 << (j % 3), t, t + (5000 if j in slow and r == 1 else 100 + int(rng.integers(0, 900)))))
        windows.append(rows)
    _windows(topo, windows, tbase_init_ns=400, tbase_rounds=max(rounds // 4, 1))
