"""GPU parity of hang location and progress rates where the regrouping of the rows can go wrong: few and many regions,
members at a region's edge, series of 2 to 200 snapshots, counters that do not fit a regrouped row, duplicates and gaps,
rings whose hops are found in LDS or by walking, and more roots than one workgroup sorts."""
import numpy as np
import pytest

from paper_2605_04478_amd import tracegen as tg
from tests import test_gpu_hang, test_gpu_rates
from tests.helpers import ring_topology

pytestmark = pytest.mark.gpu


def _cols(topo, seq, sent, recv, rng):
    """[members, channels, snapshots] states -> shuffled rows"""
    m, ch, sn = np.meshgrid(*(np.arange(k) for k in seq.shape), indexing="ij")
    comm = np.repeat(np.arange(topo.n_comms), topo.size)
    p = rng.permutation(m.size)
    flat = lambda a, dt: np.ascontiguousarray(np.broadcast_to(a, seq.shape).reshape(-1)[p].astype(dt))
    return {"snap": flat(sn, np.uint32), "rank": flat(topo.members[m], np.uint32), "comm": flat(comm[m], np.uint32),
            "channel": flat(ch, np.uint32), "seq_posted": flat(seq, np.uint64), "chunks_sent": flat(sent, np.uint32),
            "chunks_recv": flat(recv, np.uint32)}


def _random(topo, n_snap, n_ch, rng, seq0):
    shape = (int(topo.size.sum()), n_ch, n_snap)
    moves = rng.random(shape) < 0.3
    moves[rng.random(shape[0]) < 0.5, :, n_snap // 2:] = False             # half of the members stop
    seq = seq0 + np.cumsum(moves & (rng.random(shape) < 0.5), axis=2)
    cnt = np.cumsum(moves, axis=2) * 8 % 4096
    return _cols(topo, seq, cnt, cnt + (np.arange(shape[0]) % 3)[:, None, None], rng)


def _both(topo, cols, n_snap, n_ch, what, **params):
    test_gpu_hang.run_both(topo, cols, n_snap, n_ch, what=what, stall_snapshots=min(3, n_snap - 1), **params)
    test_gpu_rates.run_both(topo, cols, n_snap, n_ch, what=what)


@pytest.mark.parametrize("seq0", [0, 2**46 - 20, 2**62], ids=["small", "edge", "wide"])
@pytest.mark.parametrize("n,n_snap,n_ch", [(1, 2, 1), (63, 5, 3), (255, 64, 1), (256, 65, 2), (257, 33, 5), (513, 200, 1),
                                           (700, 130, 4), (1500, 7, 16)])
def test_sizes_and_wide_counters(n, n_snap, n_ch, seq0):
    rng = np.random.default_rng(n + n_snap)
    topo = ring_topology(n, comms=[list(range(n)), list(range(n // 2 + 1))[::-1]])
    _both(topo, _random(topo, n_snap, n_ch, rng, seq0), n_snap, n_ch, (n, n_snap, n_ch, seq0))


def test_contexts_whose_workspace_holds_anything():
    """the first hang location and the first rates of a context, and those behind a pass that does not regroup"""
    import torch

    from oracle import ccld_oracle as orc
    from paper_2605_04478_amd import ccld
    n, n_snap, n_ch = 600, 9, 2
    topo = ring_topology(n)
    rng = np.random.default_rng(3)
    new = lambda: ccld.Analyzer(topo, max_window_records=64, max_snapshot_rows=n * n_snap * n_ch, stall_snapshots=3)
    small, wide = (_random(topo, n_snap, n_ch, rng, seq0) for seq0 in (50, 2**62))
    want = [(orc.Oracle(topo, dict(stall_snapshots=3)).locate_hang(c, n_snap, n_ch), orc.Oracle(topo).progress_rates(c, n_snap, n_ch)) for c in (small, wide)]
    an = new()
    size = an.workspace.numel()
    for first in ("hang", "rates", "wide"):
        an.close()
        del an
        dirt = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda:0")
        at = dirt.data_ptr()
        torch.cuda.synchronize()
        del dirt
        an = new()
        assert an.workspace.data_ptr() == at
        for kind, k in ((first, 0),) if first != "wide" else (("hang", 1), ("hang", 0), ("rates", 1), ("rates", 0), ("rates", 1), ("hang", 0), ("hang", 1), ("rates", 0)):
            rows = an.snapshots_to_device((small, wide)[k])
            g = an.locate_hang(rows, n_snap, n_ch) if kind == "hang" else an.progress_rates(rows, n_snap, n_ch)
            o = want[k][kind == "rates"]
            assert g.status == o.status == "OK", (first, kind, k)
            for name in ("root", "pair", "comm") if kind == "hang" else ("pair", "comm"):
                ot, gt = getattr(o, name), getattr(g, name)
                assert all(np.array_equal(gt[q], ot[q]) for q in ot), (first, kind, k, name)
    an.close()


@pytest.mark.parametrize("n,n_snap", [(40, 6), (600, 70)])
def test_duplicates_gaps_and_extra_rows(n, n_snap):
    rng = np.random.default_rng(n)
    topo = ring_topology(n)
    cols = _random(topo, n_snap, 2, rng, 100)
    gap = {k: v[:-1] for k, v in cols.items()}
    extra = {k: np.concatenate([v, v[:3]]) for k, v in cols.items()}
    same = {k: np.concatenate([v[:-400], np.repeat(v[:1], 400)]) for k, v in cols.items()}
    for what, c in (("gap", gap), ("extra", extra), ("same", same)):
        _both(topo, c, n_snap, 2, what)


@pytest.mark.parametrize("n,n_snap", [(3, 9), (601, 70), (1051, 150)])
def test_a_row_too_many_in_a_region(n, n_snap):
    """regions are filled from both ends: one more row than the first or the last, smaller region has cells, and as many fewer in
    another one, or in none"""
    rng = np.random.default_rng(n)
    topo = ring_topology(n)
    cols = _random(topo, n_snap, 2, rng, 100)
    for rank in (0, n - 1):
        mine, others = np.flatnonzero(cols["rank"] == rank), np.flatnonzero(cols["rank"] == n // 2)
        _both(topo, {k: np.insert(v, n, v[mine[0]]) for k, v in cols.items()}, n_snap, 2, ("more", rank))
        moved = {k: v.copy() for k, v in cols.items()}
        for v in moved.values():
            v[others[0]] = v[mine[-1]]
        _both(topo, moved, n_snap, 2, ("moved", rank))
        _both(topo, {k: np.delete(v, mine[1]) for k, v in cols.items()}, n_snap, 2, ("fewer", rank))


@pytest.mark.parametrize("n", [64, 255, 257, 4096, 4097])
def test_hops_along_rings(n):
    topo, rng = ring_topology(n), np.random.default_rng(n)
    S, R = tg.ring_steady_state(n, n // 3, np.array([5, 9]), 1 << 20, 8)
    st = lambda a: np.repeat(np.asarray(a).astype(np.int64)[:, :, None], 4, axis=2)
    g, o = test_gpu_hang.run_both(topo, _cols(topo, np.full((n, 2, 4), 9), st(S), st(R), rng), 4, 2, what=n, stall_snapshots=2)
    assert g.n_root == 1 and int(o.pair["hops"].max()) > n // 4


@pytest.mark.parametrize("n_late", [1024, 1025])
def test_many_roots(n_late):
    n, rng = 2500, np.random.default_rng(n_late)
    topo = ring_topology(n)
    seq = np.full((n, 1, 5), 8)
    seq[rng.permutation(n)[:n_late]] = 7
    g, _ = test_gpu_hang.run_both(topo, _cols(topo, seq, np.full(seq.shape, 3), np.full(seq.shape, 3), rng), 5, 1, what=n_late, stall_snapshots=2)
    assert g.n_root == n_late


@pytest.mark.parametrize("n", [1023, 1024, 1025, 1280, 2048, 2303, 5000])
def test_rates_of_large_communicators(n):
    """the slowest member in the last or the first row of a communicator: whole steps of a workgroup over its members, and what is left"""
    topo, rng = ring_topology(n, comms=[list(range(n)), list(range(n))[::-1], list(range(n // 2))]), np.random.default_rng(n)
    cols = _random(topo, 9, 1, rng, 3)
    test_gpu_rates.run_both(topo, cols, 9, 1, what=n)
    last = cols["rank"] == n - 1
    cols["chunks_sent"][last] = cols["chunks_recv"][last] = cols["snap"][last]
    cols["seq_posted"][last] = 9 + (cols["snap"][last] > 7)
    _, o = test_gpu_rates.run_both(topo, cols, 9, 1, what=("slow", n))
    assert list(o.comm["root"][:2]) == [n - 1, n - 1]


@pytest.mark.parametrize("sizes", [[1] * 300, [2] * 131, [3, 4, 1] * 45, [1, 63, 64, 65, 2, 64, 66, 1], [65, 70], [64], [128] * 3 + [33] * 9,
                                   [2, 1] * 4100 + [65, 64, 1]],
                         ids=["ones", "pairs", "to four", "around 64", "long", "one of 64", "long first", "more than are resident"])
def test_rates_of_many_communicators(sizes):
    """communicators with some lanes of a wavefront each beside those with a workgroup each; the last workgroup partly empty, and
    more communicators than the workgroups take at once"""
    rng = np.random.default_rng(len(sizes))
    topo = ring_topology(150, comms=[list(rng.choice(150, k, replace=False)) for k in sizes])
    for snaps, ch in ((9, 2), (3, 1)):
        test_gpu_rates.run_both(topo, _random(topo, snaps, ch, rng, 3), snaps, ch, what=(len(sizes), snaps))


@pytest.mark.parametrize("n,n_snap,n_ch", [(600, 500, 16), (733, 1000, 8)])
def test_rates_of_regions_in_parts(n, n_snap, n_ch):
    """one member's series fill LDS, more members than regions: two and four parts per region, the last ones empty"""
    rng = np.random.default_rng(n)
    topo = ring_topology(n, comms=[list(range(n)), list(range(n // 2 + 1))[::-1]])
    test_gpu_rates.run_both(topo, _random(topo, n_snap, n_ch, rng, 7), n_snap, n_ch, what=(n, n_snap, n_ch))
