"""GPU parity of the grid placement where its kernels can go wrong: communicators at the edges of the lanes and fine
buckets that a collective takes, members without a record, operations in flight, values that do not fit a row, batches
that lie hours apart, and windows placed with and without communicator buckets."""
import numpy as np
import pytest

from oracle import ccld_oracle as orc
from paper_2605_04478_amd import tracegen as tg
from tests.helpers import INFLIGHT, T0, toy_cols
from tests.test_gpu_window import FAR, compare

pytestmark = pytest.mark.gpu

SIZES = {"short": [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64],
         "long": [65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1024, 1025, 2047, 2048]}
ONE_GO, BUCKETED = 0, 6_000_000       # window capacities: the records of the test, and one that takes communicator buckets


def _batch(rng, sizes, rounds, seq0, t0, missing, wide):
    """rows of `rounds` collectives per communicator, the first member always there"""
    rows = []
    for c, n in enumerate(sizes):
        for s in range(rounds + c % 3):
            t = t0 + s * 1_000_000 + c * 1000
            b = int(rng.integers(1, 1 << 30)) if not wide or s % 3 else 1 << (36 + c % 3)
            for r in range(n):
                if r and s % 2 and rng.random() < missing:
                    continue
                te = t + int(rng.integers(0, 900_000))
                tx = te + int(rng.integers(0, 5_000_000))
                u = rng.random()
                if s % 2 and u < 0.01:
                    tx = INFLIGHT
                elif wide and u < 0.05:
                    tx = te + int(rng.choice([2**32 - 3, 2**32 - 2, 2**32 - 1, 2**32, 2**40, 2**43]))
                elif wide and u < 0.08:
                    te = t0 + int(rng.choice([2**42 - 1, 2**42, 2**42 + 1, 1 - 2**42, -2**42, -2**42 - 1]))
                    tx = te + 77
                rows.append((r, c, seq0 + s, c % 6, b, te, tx))
    return rows


@pytest.mark.parametrize("cap", [ONE_GO, BUCKETED], ids=["one_go", "bucketed"])
@pytest.mark.parametrize("far_ns", [0, 2 * 3_600_000_000_000], ids=["near", "far"])
@pytest.mark.parametrize("missing,wide", [(0.0, False), (0.08, True)], ids=["full", "wide"])
@pytest.mark.parametrize("kind", ["short", "long"])
def test_grid_edges(kind, missing, wide, far_ns, cap):
    from paper_2605_04478_amd import ccld
    sizes = SIZES[kind] * (7 if kind == "short" else 1)
    topo = tg.make_topology(max(sizes), [list(range(n))[::-1] for n in sizes])
    rng = np.random.default_rng(len(sizes) + wide)
    rounds = 9 if kind == "short" else 3
    batches = [_batch(rng, sizes, rounds, 1000 + i * (rounds + 2), T0 + i * far_ns, missing, wide) for i in range(3)]
    # the counters of one communicator follow on from batch to batch: no round without a record
    nxt = [1000] * len(sizes)
    for i, rows in enumerate(batches):
        for j, r in enumerate(rows):
            rows[j] = (r[0], r[1], nxt[r[1]] + r[2] - 1000 - i * (rounds + 2)) + r[3:]
        for c in range(len(sizes)):
            nxt[c] += rounds + c % 3
    n = sum(map(len, batches))
    kw = dict(window_batches=2, tbase_init_ns=200_000, hang_threshold_ns=10**9, kmad_num=1, kmad_den=1, lag_floor_ns=50_000)
    an = ccld.Analyzer(topo, max_window_records=max(cap, n), max_batch_records=max(map(len, batches)), **kw)
    o, prev, flags = orc.Oracle(topo, kw), None, 0
    for i, rows in enumerate(batches):
        cols = toy_cols(rows)
        p = rng.permutation(len(rows))
        cols = {k: v[p] for k, v in cols.items()}
        an.ingest(an.to_device(cols))
        win = cols if prev is None else {k: np.concatenate([prev[k], cols[k]]) for k in cols}
        m = len(win["rank"])
        g, ref = an.analyze_window(FAR, n_records=m, alert_cap=m, cand_cap=2 * m, per_record=True), o.analyze_window(win, FAR)
        flags += len(ref.flag["comm"])
        compare(g, ref, *an.rank_blame(), what=f"batch{i}")
        prev = cols
    an.close()
    assert flags > 0


def _rounds(rng, n_comms, size, seq0, rounds, step, disjoint):
    """columns of `rounds` collectives of every communicator in a random order, three records left out"""
    comm, seq, slot = (x.ravel() for x in np.meshgrid(np.arange(n_comms), np.arange(rounds), np.arange(size), indexing="ij"))
    keep = rng.permutation(comm.size)[3:]
    comm, seq, slot = comm[keep], seq[keep], slot[keep]
    te = T0 + (seq0 + seq) * 1_000_000 + rng.integers(0, 500_000, keep.size)
    return {"rank": (slot + size * comm * disjoint).astype(np.uint32), "comm": comm.astype(np.uint32),
            "seq": (seq0 + seq * step).astype(np.uint64), "op": np.ones(keep.size, np.uint8),
            "bytes": np.full(keep.size, 1 << 20, np.uint64), "t_enter": te, "t_exit": te + rng.integers(1, 400_000, keep.size)}


@pytest.mark.parametrize("step", [1, 1000], ids=["grid", "sorted"])
@pytest.mark.parametrize("disjoint", [1, 0], ids=["lookup_in_lds", "many_comms_per_rank"])
def test_order_of_arrival_over_many_ingest_rounds(disjoint, step):
    """batches placed by communicator bucket: one round and many rounds per workgroup, a window that slides past one"""
    from paper_2605_04478_amd import ccld
    n_comms, size = 40, 16
    topo = tg.make_topology(size * (n_comms if disjoint else 1),
                            [[r + size * c * disjoint for r in range(size)] for c in range(n_comms)])
    rng = np.random.default_rng(3 + disjoint)
    batches, seq0 = [], 100
    for rounds in (1100, 2, 830, 3, 900):
        batches.append(_rounds(rng, n_comms, size, seq0, rounds, step, disjoint))
        seq0 += rounds * step
    an = ccld.Analyzer(topo, max_window_records=6_000_000, max_batch_records=704_000, window_batches=2)
    prev = None
    for b in batches:
        an.ingest(an.to_device(b))
        win = b if prev is None else {k: np.concatenate([prev[k], b[k]]) for k in b}
        res = an.analyze_window(FAR, n_records=len(win["rank"]), per_record=True)
        assert np.array_equal(res.per_record()["perm"], np.lexsort((win["rank"], win["seq"], win["comm"])))
        prev = b
    an.close()


@pytest.mark.parametrize("disjoint", [1, 0], ids=["lookup_in_lds", "many_comms_per_rank"])
def test_rows_that_wait_for_a_whole_line(disjoint):
    """buckets with none, a few and hundreds of records in a round of the ingest, several rounds per workgroup; batches that start in the middle
    of a line, and a window whose last line is cut by its end"""
    from paper_2605_04478_amd import ccld
    n_comms, size = 40, 3
    topo = tg.make_topology(size * (n_comms if disjoint else 1), [[r + size * c * disjoint for r in range(size)] for c in range(n_comms)])
    rng = np.random.default_rng(disjoint)
    share = 1.0 / (1 + np.arange(n_comms)) ** 3
    an = ccld.Analyzer(topo, max_window_records=6_000_011, max_batch_records=2_600_000, window_batches=2)
    prev, seq0 = None, np.full(n_comms, 7)
    for n in (2_500_001, 1_800_003, 2_599_999, 1_700_002):
        rounds = np.maximum(n / size * share / share.sum(), 1).astype(np.int64)
        comm = np.repeat(np.arange(n_comms), rounds * size)
        place = np.concatenate([np.arange(r * size) for r in rounds])
        p = rng.permutation(comm.size)[:n - n % 2]
        comm, seq, slot = comm[p], seq0[comm[p]] + place[p] // size, place[p] % size
        te = T0 + seq * 1_000 + rng.integers(0, 500, p.size)
        b = {"rank": (slot + size * comm * disjoint).astype(np.uint32), "comm": comm.astype(np.uint32), "seq": seq.astype(np.uint64),
             "op": np.ones(p.size, np.uint8), "bytes": np.full(p.size, 1 << 20, np.uint64), "t_enter": te, "t_exit": te + rng.integers(1, 400, p.size)}
        seq0 = seq0 + rounds
        an.ingest(an.to_device(b))
        win = b if prev is None else {k: np.concatenate([prev[k], b[k]]) for k in b}
        res = an.analyze_window(FAR, n_records=len(win["rank"]), per_record=True)
        order = np.lexsort((win["rank"], win["seq"], win["comm"]))
        assert np.array_equal(res.per_record()["perm"], order)
        seg = res.seg
        first = seg["first"][:res.n_seg]
        te, dur = win["t_enter"][order], (win["t_exit"] - win["t_enter"])[order]
        assert np.array_equal(np.minimum.reduceat(te, first), seg["enter_min"]) and np.array_equal(np.maximum.reduceat(dur, first), seg["dur_max"])
        prev = b
    an.close()


def _large(sizes, rounds, drop, seed):
    """device columns of rounds[c] collectives of every communicator c in a random order, most of the first `drop` left out, and what follows
    from them per collective in table order: records, earliest arrival, longest duration"""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    i64 = dict(dtype=torch.int64, device="cuda")
    size, first = torch.tensor(sizes, **i64), torch.tensor(np.concatenate([[0], np.cumsum(sizes)[:-1]]), **i64)
    rounds = torch.tensor(rounds, **i64)
    comm = torch.repeat_interleave(torch.arange(len(sizes), **i64), rounds * size)
    place = torch.arange(comm.numel(), **i64) - torch.repeat_interleave(torch.cumsum(rounds * size, 0) - rounds * size, rounds * size)
    row = torch.repeat_interleave(torch.cumsum(rounds, 0) - rounds, rounds * size) + place // size[comm]
    keep = torch.randperm(comm.numel(), generator=gen, device="cuda")
    keep = keep[(keep >= drop) | (place[keep] % size[comm[keep]] == 0)]        # (the first member of every collective stays)
    comm, place, row = comm[keep], place[keep], row[keep]
    te = T0 + row * 1000 + torch.randint(0, 500, row.shape, generator=gen, device="cuda")
    dur = torch.randint(1, 400, row.shape, generator=gen, device="cuda")
    n_seg = int(rounds.sum())
    want = (torch.bincount(row, minlength=n_seg), torch.full((n_seg,), 2**62, **i64).scatter_reduce_(0, row, te, "amin"),
            torch.zeros(n_seg, **i64).scatter_reduce_(0, row, dur, "amax"))
    cols = {"rank": (first[comm] + place % size[comm]).int(), "comm": comm.int(), "seq": 5 + place // size[comm],
            "op": torch.ones(comm.numel(), dtype=torch.uint8, device="cuda"), "bytes": torch.full((comm.numel(),), 64, **i64), "t_enter": te, "t_exit": te + dur}
    return cols, want


# 192 communicators, two to a coarse bucket: such of 2,048 cells per fine bucket and of fewer, some with so many fine buckets that they
# leave as runs beside others
@pytest.mark.parametrize("mix", ["even", "odd", "skewed"])
def test_largest_windows_leave_in_whole_lines(mix):
    from paper_2605_04478_amd import ccld
    n, n_comms = 51_000_000, 192
    sizes = {"even": [8] * n_comms, "odd": [3 + (5 * c) % 62 for c in range(n_comms)], "skewed": [64] * n_comms}[mix]
    share = np.ones(n_comms) if mix != "skewed" else 1.0 / (1 + np.arange(n_comms) % 24) ** 2
    rounds = np.maximum(n * share / share.sum() / sizes, 1).astype(int) + np.arange(n_comms) % 3
    cols, want = _large(sizes, rounds, 0 if mix == "even" else 1001, len(mix))
    off = np.concatenate([[0], np.cumsum(sizes)])
    topo = tg.make_topology(int(off[-1]), [list(range(off[c], off[c + 1])) for c in range(n_comms)])
    n = cols["comm"].numel()
    assert n // 256 >= 64 * 3072
    an = ccld.Analyzer(topo, max_window_records=n)
    an.profile_enable(True)
    bufs = an.alloc_window_result(n, seg_cap=int(rounds.sum()), flag_cap=1024, group_cap=1 << 18)
    for again in range(2):
        an.reset_window()
        an.ingest(cols)
        res = an.analyze_window(FAR, buffers=bufs)
        assert res.n_seg == rounds.sum() and res.status in ("OK", "TRUNCATED", "W_TRUNCATED")
        seg = res.dev["seg"].view(21, -1)
        for name, w in zip(("n", "enter_min", "dur_max"), want):
            assert bool((seg[ccld.SEG_COLS.index(name)] == w).all()), (mix, again, name)
    assert an.profile_read()[0]["sort_hist"][1] == 0                  # it stayed on the grid
    # a record twice; one a hundred thousand times, more than a fine bucket's counts of rows can tell; in a context that has analysed
    # the same layout and in a new one
    for copies in (2, 100_000):
        bad = {k: v.clone() for k, v in cols.items()}
        at = slice(1000, 1000 + copies)
        for k in bad:
            bad[k][at] = bad[k][999]
        for fresh in (False, True):
            if fresh:
                an.close()
                an = ccld.Analyzer(topo, max_window_records=n)
            an.reset_window()
            an.ingest(bad)
            assert an.analyze_window(FAR, buffers=bufs).status == "E_DUPLICATE_KEY"
    an.reset_window()
    an.ingest(cols)
    assert an.analyze_window(FAR, buffers=bufs).n_seg == rounds.sum()
    an.close()


def _edited(cols, seed):
    """some of the records late, of another size, in flight or of full width"""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n = cols["comm"].numel()
    at = lambda k: torch.randint(0, n, (k,), generator=gen, device="cuda")
    late, slow, wide, far, other, open_ = at(4000), at(4000), at(800), at(200), at(400), at(100)
    cols["t_enter"][late] += 100_000
    cols["t_exit"][late] += 100_000
    cols["t_exit"][slow] += 200_000
    cols["t_exit"][wide] += 2**32
    cols["t_enter"][far] -= 2**42
    cols["bytes"][other] = 2**37 + 5
    cols["t_exit"][open_] = INFLIGHT
    return cols


LINES_FROM = 256 * 64 * 3072          # records of a window whose rows leave the partition in whole lines
LINES_SIZES = {
    "even": [8] * 192, "odd": [3 + (5 * c) % 62 for c in range(192)],
    # communicators whose rounds are too few for fine buckets that start on lines (257, 301, 701), beside such as are enough
    "long": [(64, 257, 65, 300, 301, 129, 255, 701, 700, 33, 7, 128)[c % 12] for c in range(192)],
    # every eighth coarse bucket holds so few records that they leave as runs
    "sparse": [16 + c % 3 for c in range(192)],
}


@pytest.mark.parametrize("mix", list(LINES_SIZES))
def test_whole_lines_and_runs_give_the_same_tables(mix):
    """A sliding window of three batches whose rows leave in whole lines, and the same with the order of the records, with which they leave as
    runs from a grid that does not start on lines: rounds of the partition that cross pieces, a circular window that wraps, members
    missing here and there, late records, rows of full width, and operations in flight; every table of both is the same."""
    import torch
    from paper_2605_04478_amd import ccld
    sizes = LINES_SIZES[mix]
    n_comms = len(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)])
    topo = tg.make_topology(int(off[-1]), [list(range(off[c], off[c + 1])) for c in range(n_comms)])
    share = np.where((mix == "sparse") & (np.arange(n_comms) // 2 % 8 == 3), 0.0, 1.0) / sizes
    W, batches, seq0 = 3, [], np.zeros(n_comms, np.int64)
    for i, n in enumerate((17_500_000, 17_800_003, 17_600_001, 17_550_000, 17_700_005)):
        rounds = np.maximum(n * share / (share * sizes).sum(), 3).astype(int) + (np.arange(n_comms) + i) % 3
        cols, _ = _large(sizes, rounds, 0 if mix == "even" else 500_000, 10 * i + len(mix))
        cols["seq"] += torch.from_numpy(seq0).cuda()[cols["comm"].long()]
        later = int(rounds.max()) * 2000
        for k in ("t_enter", "t_exit"):
            cols[k] += i * later
        seq0 += rounds
        batches.append(_edited(cols, i))
    count = [b["comm"].numel() for b in batches]
    cap = max(sum(count[i:i + W]) for i in range(len(count) - W + 1))
    kw = dict(window_batches=W, lag_floor_ns=10_000, hang_threshold_ns=10**9, tbase_init_ns=1000)
    an = [ccld.Analyzer(topo, max_window_records=cap, max_batch_records=max(count), **kw) for _ in range(2)]
    bufs = [a.alloc_window_result(cap, seg_cap=cap // 2, flag_cap=1 << 20, group_cap=1 << 18, cand_cap=1 << 20, per_record=r) for a, r in zip(an, (False, True))]
    for a in an:
        a.profile_enable(True)
    for i, b in enumerate(batches):
        for a in an:
            a.ingest(b)
        if i + 1 < W:
            continue
        n = sum(count[i + 1 - W:i + 1])
        assert n >= LINES_FROM
        g, ref = (a.analyze_window(FAR, buffers=x) for a, x in zip(an, bufs))
        assert g.status == ref.status == "OK" and g.n_records == ref.n_records == n
        assert (g.n_seg, g.n_flag, g.n_group, g.n_alert, g.n_cand) == (ref.n_seg, ref.n_flag, ref.n_group, ref.n_alert, ref.n_cand)
        assert g.n_flag > 1000 and g.n_alert > 100 and g.n_seg >= n // 701
        for name, m in (("seg", g.n_seg), ("flag", g.n_flag), ("group", g.n_group), ("alert", g.n_alert), ("cand", g.n_cand)):
            x, y = (r.dev[name].view(-1, r.caps[name])[:, :m] for r in (g, ref))
            assert bool((x == y).all()), (mix, i, name)
        (blame, order), (blame2, order2) = (a.rank_blame() for a in an)
        assert all(np.array_equal(blame[k], blame2[k]) for k in blame) and np.array_equal(order, order2), (mix, i)
    for a in an:
        assert a.profile_read()[0]["sort_hist"][1] == 0
        a.close()


@pytest.mark.parametrize("mix", ["even", "odd"])
@pytest.mark.parametrize("gone", [False, True], ids=["on_the_grid", "a_round_gone"])
def test_rounds_that_nobody_recorded_in_whole_lines(mix, gone):
    """a twentieth of the records missing, so that the rounds of most fine buckets are looked at one by one, filled from both ends: the window stays
    on the grid; with the first, one inner or the last round of a communicator's second fine bucket gone too, it is sorted"""
    from paper_2605_04478_amd import ccld
    sizes = LINES_SIZES[mix]
    n_comms = len(sizes)
    rounds = np.full(n_comms, 53_500_000 // sum(sizes) + 1)
    off = np.concatenate([[0], np.cumsum(sizes)])
    topo = tg.make_topology(int(off[-1]), [list(range(off[c], off[c + 1])) for c in range(n_comms)])
    cols, (want_n, _, _) = _large(sizes, rounds, 3_000_000, 5)
    n = cols["comm"].numel()
    assert 0.045 < 1 - n / (rounds * sizes).sum() < 0.06 and n >= LINES_FROM + 5000
    an = ccld.Analyzer(topo, max_window_records=n)
    bufs = an.alloc_window_result(n, seg_cap=int(rounds.sum()), flag_cap=1024, group_cap=1 << 18)
    c = 100
    rpb = 2048 // sizes[c] // 8 * 8
    for q in ((rpb, rpb + 77 % rpb, 2 * rpb - 1) if gone else (None,)):
        keep = slice(None) if q is None else ~((cols["comm"] == c) & (cols["seq"] == 5 + q))
        b = {k: v[keep] for k, v in cols.items()}
        an.profile_enable(True)
        sorts = an.profile_read()[0]["sort_hist"][1]
        an.reset_window()
        an.ingest(b)
        res = an.analyze_window(FAR, buffers=bufs)
        assert res.n_seg == rounds.sum() - (q is not None) and res.status in ("OK", "W_TRUNCATED"), (q, res.status)
        assert (an.profile_read()[0]["sort_hist"][1] > sorts) == gone
        have, row = res.dev["seg"].view(21, -1)[ccld.SEG_COLS.index("n")], int(rounds[:c].sum())
        if q is None:
            assert bool((have == want_n).all())
        else:
            assert bool((have[:row + q] == want_n[:row + q]).all()) and bool((have[row + q:res.n_seg] == want_n[row + q + 1:]).all())
    an.close()


SHORT_SIZES = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64]


@pytest.mark.parametrize("per_record", [True, False], ids=["per_record", "tables"])
@pytest.mark.parametrize("n_comms", [620, 1300], ids=["eight_wavefronts", "four_wavefronts"])
def test_buckets_that_are_full_but_for_one_record(n_comms, per_record):
    """Fine buckets with a record in every cell, beside such where one operation is in flight, one row is of full width or at an edge of it, or one
    record is missing, in the first, an inner or the last cell, in the layouts whose statistics take full buckets by a path of their own"""
    from paper_2605_04478_amd import ccld
    rng = np.random.default_rng(n_comms)
    sizes = [SHORT_SIZES[c % 16] for c in range(n_comms)]
    topo = tg.make_topology(64, [list(range(n)) for n in sizes])
    rows = []
    for c, n in enumerate(sizes):
        K = 4 + c % 5
        odd, where = c // 16 % 9, (0, K * n - 1, int(rng.integers(K * n)))[c // 7 % 3]
        for s in range(K):
            t = T0 + s * 10**7 + c * 1000
            for r in range(n):
                te = t + int(rng.integers(0, 50_000)) + (10**6 if rng.random() < 0.02 else 0)
                tx, nb = te + int(rng.integers(1, 200_000)), 1 << 20
                if s * n + r == where:
                    if odd == 1:
                        tx = INFLIGHT
                    elif odd in (2, 3, 4, 5):
                        tx = te + (2**32 - 3, 2**32 - 2, 2**30, 2**30 - 1)[odd - 2]
                    elif odd == 6:
                        te = te - 2**42
                    elif odd == 7:
                        nb = 2**37
                    elif odd == 8 and n > 1:
                        continue
                rows.append((r, c, 3 + s, 1, nb, te, tx))
    cols = toy_cols([rows[i] for i in rng.permutation(len(rows))])
    n = len(rows)
    assert n // 2048 + n_comms // 2 > 256 and (n // 2048 + n_comms // 2 <= 512) == (n_comms == 620)
    kw = dict(lag_floor_ns=100_000, tbase_init_ns=200_000, hang_threshold_ns=10**9)
    an = ccld.Analyzer(topo, max_window_records=n, **kw)
    an.profile_enable(True)
    an.ingest(an.to_device(cols))
    g = an.analyze_window(FAR, n_records=n, alert_cap=n, cand_cap=2 * n, per_record=per_record)
    ref = orc.Oracle(topo, kw).analyze_window(cols, FAR)
    compare(g, ref, *an.rank_blame(), per_record=per_record, what=n_comms)
    assert an.profile_read()[0]["sort_hist"][1] == 0 and g.n_flag > 100 and g.n_alert > 30
    an.close()


@pytest.mark.parametrize("floor_ns", [0, -1, -2**31, -2**40, 5, 2**31 - 2, 2**31 - 1, 2**31, 2**40])
@pytest.mark.parametrize("many", [1, 40], ids=["few", "many"])
def test_floors_of_the_lag_at_the_edges_of_32_bits(floor_ns, many):
    """a collective is done with when no lag is above the floor: floors of zero, below it, and beyond what a lag can be"""
    from paper_2605_04478_amd import ccld
    rng = np.random.default_rng(9)
    sizes = [2, 4, 8, 33, 64, 65, 100, 128, 129, 200, 256, 257, 400, 512, 513] * many
    topo = tg.make_topology(max(sizes), [list(range(n)) for n in sizes])
    rows = []
    for c, n in enumerate(sizes):
        for s in range(3):
            t = T0 + s * 10**10 + c * 1000
            te = t + rng.integers(0, (2, 1000, 2**29)[s], n)
            te[rng.random(n) < 0.05] += 2**29
            tx = te + rng.integers(1, 100, n)
            tx[rng.random(n) < 0.05] += 2**28
            rows += [(r, c, s, 1, 64, int(a), int(b)) for r, (a, b) in enumerate(zip(te, tx))]
    cols = toy_cols([rows[i] for i in rng.permutation(len(rows))])
    n = len(rows)
    for kmad in (0, 9):
        kw = dict(lag_floor_ns=floor_ns, kmad_num=kmad, kmad_den=2)
        an = ccld.Analyzer(topo, max_window_records=n, **kw)
        an.ingest(an.to_device(cols))
        g = an.analyze_window(FAR, n_records=n)
        ref = orc.Oracle(topo, kw).analyze_window(cols, FAR)
        compare(g, ref, *an.rank_blame(), per_record=False, what=(floor_ns, kmad))
        assert (g.n_flag > 0) == (floor_ns < 2**31 - 2)
        an.close()


GAP_SIZES = [1, 2, 3, 31, 64, 65, 700, 2048]


@pytest.mark.parametrize("comm,place", [(0, 1), (0, 2047), (0, 2048), (0, 2078), (1, 1023), (1, 1024), (2, 681), (2, 700), (3, 66), (4, 31),
                                        (4, 40), (5, 30), (6, 1), (7, 2), (None, 0), (None, 1)])
def test_rounds_that_nobody_recorded_in_large_layouts(comm, place):
    """Layouts of more than 4,096 fine buckets, where a round without any record is looked for before the statistics: in the
    first and last rounds of fine buckets and words of their bitmaps, for communicators of 1 to 2,048 members; and
    windows that only lack single records, which stay on the grid."""
    from paper_2605_04478_amd import ccld
    rng = np.random.default_rng(place)
    many = 3_500
    R = 4096
    comms = [list(range(n)) for n in GAP_SIZES] + [[int(x) for x in rng.choice(R, 2, replace=False)] for _ in range(many)]
    rounds = [2100, 1100, 720, 140, 70, 64, 6, 4] + [20] * many
    cols = {k: [] for k in ("rank", "comm", "seq", "t_enter")}
    for c, (mem, n) in enumerate(zip(comms, rounds)):
        q = np.repeat(np.arange(n), len(mem))
        keep = np.ones(q.size, dtype=bool)
        if comm is None and place and len(mem) > 1:          # a record missing here and there, never a whole round
            keep = (np.tile(np.arange(len(mem)), n) == q % len(mem)) | (rng.random(q.size) > 0.05)
        if c == comm:
            keep = q != place
        cols["rank"].append(np.tile(mem, n)[keep])
        cols["comm"].append(np.full(keep.sum(), c))
        cols["seq"].append(10 + q[keep])
        cols["t_enter"].append(T0 + q[keep] * 1_000_000 + rng.integers(0, 900_000, keep.sum()))
    cols = {k: np.concatenate(v) for k, v in cols.items()}
    n = cols["rank"].size
    cols["t_exit"] = cols["t_enter"] + rng.integers(0, 3_000_000, n)
    p = rng.permutation(n)
    dt = {"rank": np.uint32, "comm": np.uint32, "seq": np.uint64, "t_enter": np.int64, "t_exit": np.int64}
    cols = {k: v[p].astype(dt[k]) for k, v in cols.items()}
    cols["op"], cols["bytes"] = np.zeros(n, dtype=np.uint8), np.full(n, 1 << 20, dtype=np.uint64)
    topo = tg.make_topology(R, comms)
    an = ccld.Analyzer(topo, max_window_records=4_000_000, max_batch_records=n)
    an.ingest(an.to_device(cols))
    an.profile_enable(True)
    g, ref = an.analyze_window(FAR, n_records=n, per_record=True), orc.Oracle(topo).analyze_window(cols, FAR)
    compare(g, ref, *an.rank_blame(), what=f"gap at {comm}, {place}")
    times, _ = an.profile_read()
    assert (times["sort_hist"][1] > 0) == (comm is not None)
    an.close()


def _one(topo, cols, cap):
    """one batch in a context of a larger window"""
    from paper_2605_04478_amd import ccld
    n = cols["rank"].size
    an = ccld.Analyzer(topo, max_window_records=cap, max_batch_records=n)
    an.ingest(an.to_device(cols))
    g = an.analyze_window(FAR, n_records=n, per_record=True)
    compare(g, orc.Oracle(topo).analyze_window(cols, FAR), *an.rank_blame(), what=(topo.n_comms, n))
    an.close()


@pytest.mark.parametrize("n_comms,n", [(32, 256 * 2048), (33, 248 * 2048), (33, 248 * 2048 + 1)])
def test_counts_summed_by_the_placement_or_scanned(n_comms, n):
    """as many words of counts (communicator buckets times workgroups) as every placement workgroup sums for itself, fewer, and more"""
    topo = tg.make_topology(64, [[c, c + 1, c + 9] for c in range(n_comms)])
    per = n // (3 * n_comms)
    i = np.random.default_rng(n).permutation(3 * n_comms * (per + 1))[:n]
    comm, seq = i // 3 % n_comms, i // (3 * n_comms)
    rng = np.random.default_rng(n_comms)
    te = T0 + seq * 10**6 + rng.integers(0, 1000, n)
    te[rng.random(n) < 0.001] += 10**5
    cols = {"rank": np.concatenate([topo.members_of(c) for c in range(n_comms)])[3 * comm + i % 3].astype(np.uint32), "comm": comm.astype(np.uint32),
            "seq": seq.astype(np.uint64), "op": np.ones(n, np.uint8), "bytes": np.full(n, 64, np.uint64), "t_enter": te, "t_exit": te + 5 * 10**5}
    _one(topo, cols, 28_000_000)


def test_one_batch_of_few_buckets_and_four_counting_workgroups_each():
    """2^23 records and more in one batch, a communicator that the grid does not take, eight buckets"""
    n = 2100
    topo = tg.make_topology(n, [list(range(n))] + [list(range(300 * c, 300 * c + 300)) for c in range(7)])
    rounds = 1998
    q = np.repeat(np.arange(rounds), 2 * n)
    rank = np.tile(np.concatenate([np.arange(n)] * 2), rounds)
    comm = np.tile(np.concatenate([np.zeros(n, np.int64), 1 + np.arange(n) // 300]), rounds)
    rng = np.random.default_rng(8)
    te = T0 + q * 10**6 + rng.integers(0, 1000, q.size)
    te[rng.integers(0, q.size, 500)] += 10**5
    p = rng.permutation(q.size)
    cols = {"rank": rank.astype(np.uint32), "comm": comm.astype(np.uint32), "seq": q.astype(np.uint64), "op": np.ones(q.size, np.uint8),
            "bytes": np.full(q.size, 64, np.uint64), "t_enter": te, "t_exit": te + 5 * 10**5}
    assert q.size >= 1 << 23
    _one(topo, {k: v[p] for k, v in cols.items()}, 26_000_000)
