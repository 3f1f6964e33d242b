"""GPU parity of the end of an analysis (groups, flags, blame order and alerts side by side, then group table and report) where it
can go wrong: alerts around the number and the communicators that it lists itself, flags around the fine buckets of a thread and of
a workgroup, more ranks than it orders, and of the calls that report from their last kernel when they follow one another."""
import numpy as np
import pytest

from oracle import ccld_oracle as orc
from paper_2605_04478_amd import tracegen as tg
from tests.helpers import INFLIGHT, T0, ring_topology, toy_cols
from tests.test_gpu_frames import both
from tests.test_gpu_window import FAR, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("step", [1, 10**6], ids=["grid", "sorted"])
@pytest.mark.parametrize("n_alert", [1, 7, 8, 9, 40])
def test_alerts_of_every_class(n_alert, step):
    """collectives that some member has not entered, that some finished, that all hang in; sizes around a wavefront"""
    sizes = [2, 3, 63, 64, 65, 130, 700]
    topo = tg.make_topology(700, [list(range(n))[::-1] for n in sizes])
    rng = np.random.default_rng(n_alert)
    rows = []
    for c, n in enumerate(sizes):
        hung = {int(s) for s in rng.permutation(9)[:(n_alert + len(sizes) - 1 - c) // len(sizes)]}
        for s in range(9):
            cls = int(rng.integers(0, 3)) if s in hung else -1
            for r in range(n):
                te = T0 + s * 10**9 + int(rng.integers(0, 10**6))
                tx = te + 10**6
                if cls == 0 and r % 3 == 1 or cls >= 0 and r == 0 and cls != 1:
                    if cls == 0 and r % 3 == 1:
                        continue
                    tx = INFLIGHT
                if cls == 2 or cls == 1 and r % 2:
                    tx = INFLIGHT
                rows.append((r, c, 5 + s * step, 1, 1 << 20, te, tx))
    p = np.random.default_rng(1).permutation(len(rows))
    cols = {k: v[p] for k, v in toy_cols(rows).items()}
    g, o = run_both(topo, cols, hang_threshold_ns=10**9, what=(n_alert, step))
    assert g.n_alert == n_alert


@pytest.mark.parametrize("step", [1, 10**6], ids=["grid", "sorted"])
@pytest.mark.parametrize("n", [2048, 2049])
@pytest.mark.parametrize("n_alert", [1, 8, 9])
def test_alerts_of_large_communicators(n_alert, n, step):
    """the most members whose candidates a wavefront marks, and one more, which is listed by the launches of longer lists"""
    topo = tg.make_topology(n, [list(range(n))[::-1], [5, 3, 4]])
    rng = np.random.default_rng(n_alert)
    q, r = np.repeat(np.arange(10), n), np.tile(np.arange(n), 10)
    te = T0 + q * 10**9 + rng.integers(0, 10**6, q.size)
    tx, keep = te + 10**6, np.ones(q.size, bool)
    for a in range(n_alert):               # not entered by the last and by some others, finished by some, hung in by all
        on = q == a
        some = on & ((r % 5 == 1) | (r == n - 1))
        if a % 3 == 0:
            keep &= ~some
        tx[on & ~some if a % 3 == 1 else on] = INFLIGHT
    more = np.arange(3, 6)
    cols = {"rank": np.concatenate([r[keep], more]), "comm": np.concatenate([0 * r[keep], 0 * more + 1]), "seq": np.concatenate([q[keep] * step, 0 * more]),
            "t_enter": np.concatenate([te[keep], T0 + more]), "t_exit": np.concatenate([tx[keep], T0 + 9 + more])}
    cols = {**{k: v.astype(np.uint32 if k in ("rank", "comm") else np.uint64 if k == "seq" else np.int64) for k, v in cols.items()},
            "op": np.ones(keep.sum() + 3, np.uint8), "bytes": np.full(keep.sum() + 3, 64, np.uint64)}
    p = rng.permutation(keep.sum() + 3)
    g, o = run_both(topo, {k: v[p] for k, v in cols.items()}, hang_threshold_ns=10**9, what=(n_alert, n, step))
    assert g.n_alert == n_alert and g.n_cand > n // 5


def test_truncated_alert_tables():
    from paper_2605_04478_amd import ccld
    topo = ring_topology(6)
    rows = [(r, 0, s, 1, 64, T0 + s, INFLIGHT if r < 2 else T0 + s + 9) for s in range(5) for r in range(6)]
    cols = toy_cols(rows)
    ref = orc.Oracle(topo, dict(hang_threshold_ns=10)).analyze_window(cols, FAR)
    for alert_cap, cand_cap in ((5, 20), (3, 20), (5, 7), (1, 1)):
        an = ccld.Analyzer(topo, max_window_records=30, hang_threshold_ns=10)
        an.ingest(an.to_device(cols))
        g = an.analyze_window(FAR, n_records=30, alert_cap=alert_cap, cand_cap=cand_cap)
        assert (g.n_alert, g.n_cand) == (5, 20) and g.status == ("OK" if (alert_cap, cand_cap) == (5, 20) else "W_TRUNCATED")
        for k in ref.alert:
            assert np.array_equal(g.alert[k], ref.alert[k][:alert_cap]), k
        assert np.array_equal(g.cand, ref.cand[:cand_cap])
        an.close()


@pytest.mark.parametrize("buckets", [1, 8, 9, 16, 17, 63, 64, 65, 128, 129, 257])
def test_flags_in_every_bucket(buckets):
    """one communicator of 1,024 members (two rounds in a fine bucket); eight buckets to a thread of the scan, sixteen to a workgroup
    of the list, 64 probed at a time"""
    n = 1024
    topo = ring_topology(n)
    rng = np.random.default_rng(buckets)
    q = np.repeat(np.arange(2 * buckets), n)
    rank = np.tile(np.arange(n), 2 * buckets)
    te = T0 + q * 10**9 + rng.integers(0, 1000, q.size)
    te[rng.integers(0, q.size, 5 * buckets)] += 10**7
    p = rng.permutation(q.size)
    cols = {"rank": rank.astype(np.uint32), "comm": np.zeros(q.size, np.uint32), "seq": q.astype(np.uint64), "op": np.ones(q.size, np.uint8),
            "bytes": np.full(q.size, 64, np.uint64), "t_enter": te, "t_exit": T0 + q * 10**9 + 5 * 10**7 + rng.integers(0, 1000, q.size)}
    g, o = run_both(topo, {k: v[p] for k, v in cols.items()}, what=buckets)
    assert g.n_flag >= 4 * buckets


@pytest.mark.parametrize("first,pairs,last", [(1, 0, 1), (63, 1, 2), (65, 0, 70), (130, 300, 66), (398, 3300, 398), (398, 3300, 399), (500, 3400, 333)])
def test_flags_far_apart_and_close_together(first, pairs, last):
    """the fine buckets of two rings of 1,025 members (a round each) around those of pairs, which have no flag: runs of 64 flags within a
    bucket, in as many buckets and over thousands of them, and numbers of buckets on both sides of what a workgroup scans"""
    n = 1025
    topo = tg.make_topology(n, [list(range(n))] + [[c % 1000, c % 1000 + 1 + c // 1000] for c in range(pairs)] + [list(range(n))[::-1]])
    rng = np.random.default_rng(first + last)
    rows = [(np.zeros(first * n, np.int64), np.repeat(np.arange(first), n), np.tile(np.arange(n), first)),
            (np.repeat(np.arange(1, pairs + 1), 2), np.zeros(2 * pairs, np.int64), np.concatenate([topo.members_of(1 + c) for c in range(pairs)] + [np.zeros(0, np.int64)])),
            (np.full(last * n, pairs + 1), np.repeat(np.arange(last), n), np.tile(np.arange(n), last))]
    comm, seq, rank = (np.concatenate(x) for x in zip(*rows))
    te = T0 + seq * 10**9 + rng.integers(0, 1000, comm.size)
    late = np.zeros(comm.size, bool)
    late[rng.integers(0, n, min(first, 70)) + np.arange(min(first, 70)) * n] = True                     # one flag a bucket
    late[(comm == 0) & (seq == first - 1) & (rank % 7 == 3)] = True                                     # 146 in one
    late[(comm == pairs + 1) & (seq == 0) & (rank % 16 == 1)] = True                                    # 64
    late[(comm == pairs + 1) & (seq == last - 1) & (rank % 3 == 0)] = True                              # 342, in the last bucket
    te[late] += 10**7
    p = rng.permutation(comm.size)
    cols = {"rank": rank.astype(np.uint32), "comm": comm.astype(np.uint32), "seq": seq.astype(np.uint64), "op": np.ones(comm.size, np.uint8),
            "bytes": np.full(comm.size, 64, np.uint64), "t_enter": te, "t_exit": T0 + seq * 10**9 + 5 * 10**7 + rng.integers(0, 1000, comm.size)}
    g, o = run_both(topo, {k: v[p] for k, v in cols.items()}, what=(first, pairs, last))
    assert g.n_flag == int(late.sum())


@pytest.mark.parametrize("n_ranks", [511, 512, 2048, 2049, 16384, 16385])
def test_blame_order_of_many_ranks(n_ranks):
    topo = tg.make_topology(n_ranks, [list(range(i, min(i + 8, n_ranks))) for i in range(0, n_ranks, 8)])
    rng = np.random.default_rng(n_ranks)
    r = np.tile(np.arange(n_ranks), 3)
    q = np.repeat(np.arange(3), n_ranks)
    te = T0 + q * 10**9 + rng.integers(0, 1000, r.size)
    te[rng.random(r.size) < 0.1] += 10**7
    cols = {"rank": r.astype(np.uint32), "comm": (r // 8).astype(np.uint32), "seq": q.astype(np.uint64), "op": np.ones(r.size, np.uint8),
            "bytes": np.full(r.size, 64, np.uint64), "t_enter": te, "t_exit": te + 5 * 10**7}
    run_both(topo, cols, what=n_ranks)


@pytest.mark.parametrize("n_ranks", [1, 65, 16384, 16385])
def test_windows_without_records(n_ranks):
    from paper_2605_04478_amd import ccld
    topo = ring_topology(n_ranks)
    an = ccld.Analyzer(topo, max_window_records=2 * n_ranks)
    rows = toy_cols([(r, 0, 1, 1, 64, T0 + (10**7 if r % 50 == 7 else r % 13), T0 + 10**8) for r in range(n_ranks)])
    for cols in ({k: v[:0] for k, v in rows.items()}, rows, None, {k: v[:0] for k, v in rows.items()}):
        an.reset_window()
        if cols is not None:
            an.ingest(an.to_device(cols))
        g = an.analyze_window(FAR, n_records=n_ranks, per_record=True)
        ref = orc.Oracle(topo).analyze_window(cols if cols is not None else {k: v[:0] for k, v in rows.items()}, FAR)
        blame, order = an.rank_blame()
        assert g.status == ref.status == "OK" and g.n_seg == len(ref.seg["comm"]) and g.n_flag == len(ref.flag["comm"])
        assert np.array_equal(order, ref.order) and all(np.array_equal(blame[k], ref.blame[k]) for k in ref.blame)
    an.close()


def test_calls_that_report_from_their_last_kernel_in_turn():
    """analysis, blame, chains, hang location, rates and frames on one context: each leaves the counters as the next needs them"""
    from paper_2605_04478_amd import ccld
    from tests.test_oracle_hang import snap_rows
    tr = tg.generate(tg.config1(n_slots=60))
    topo = tr.topo
    o = orc.Oracle(topo)
    m = int(topo.size.sum())
    an = ccld.Analyzer(topo, max_window_records=tr.n, max_snapshot_rows=max(m * 4, 64 * topo.n_ranks))
    snaps = snap_rows(topo, 4, 1, lambda s, c, q, ch: (3, 5 + s, 5) if q else (2, 9, 9))
    bad = {k: np.concatenate([v[:-1], v[:1]]) for k, v in snaps.items()}
    frames = np.zeros(topo.n_ranks, dtype=tg.FRAME_DTYPE)
    frames["n_channels"] = 1
    frames["block"]["ext"][:, :1], frames["block"]["comm"][:, :1] = 1, 0
    decoder = orc.Oracle(topo)
    decoder.frames_begin(1)
    call = 0
    for i in range(4):
        an.reset_window()
        an.ingest(an.to_device(tr.cols))
        g, ref = an.analyze_window(FAR, n_records=tr.n, per_record=True), o.analyze_window(tr.cols, FAR)
        compare(g, ref, *an.rank_blame(), what=i)
        chain, per_rank = o.flag_chains(tr.cols, ref)
        for _ in range(2):
            st, gc, gr = an.flag_chains(g)
            assert st == "OK" and all(np.array_equal(gc[k], chain[k]) for k in chain) and all(np.array_equal(gr[k], per_rank[k]) for k in per_rank)
        for rows, status in ((snaps, "OK"), (bad, "E_DUPLICATE_KEY"), (snaps, "OK")):
            h = an.locate_hang(an.snapshots_to_device(rows), 4, 1)
            r = an.progress_rates(an.snapshots_to_device(rows), 4, 1)
            assert (h.status, r.status) == (status, status)
            if status == "OK":
                want, rate = orc.Oracle(topo).locate_hang(rows, 4, 1), orc.Oracle(topo).progress_rates(rows, 4, 1)
                for got, ref_of in ((h, want), (r, rate)):
                    for name in ("root", "pair", "comm") if got is h else ("pair", "comm"):
                        table, expected = getattr(got, name), getattr(ref_of, name)
                        assert all(np.array_equal(table[k], expected[k]) for k in expected), (i, status, name)
            call += 1
            frames["block"]["counter"][:, 0] = call
            frames["block"]["count"][:, 0, 0] = np.arange(topo.n_ranks)[:, None] * [3, 5] + call
            both(an, decoder, frames.view(np.uint8).reshape(topo.n_ranks, -1), np.arange(topo.n_ranks, dtype=np.uint32), call, 1, on_device=bool(call % 2), what=call)
        blame, order = an.rank_blame()
        assert np.array_equal(order, ref.order) and all(np.array_equal(blame[k], ref.blame[k]) for k in ref.blame)
    an.close()


def test_snapshots_of_more_regions_than_the_pass_before():
    """hang location and rates on one context over few, many and few snapshots: a pass leaves the fills of every region clear"""
    from paper_2605_04478_amd import ccld
    n = 1024
    topo = tg.make_topology(n, [list(range(i, i + 16)) for i in range(0, n, 16)] + [list(range(i, n, 64)) for i in range(64)])
    m = int(topo.size.sum())
    comm = np.repeat(np.arange(topo.n_comms), topo.size)
    rank = np.concatenate([topo.members_of(c) for c in range(topo.n_comms)])
    rng = np.random.default_rng(5)
    an = ccld.Analyzer(topo, max_window_records=64, max_snapshot_rows=m * 64)
    for n_snap, n_ch in ((2, 1), (16, 4), (2, 1), (7, 2), (16, 4)):
        i = rng.permutation(m * n_snap * n_ch)
        q, s, ch = i // (n_snap * n_ch), i % n_snap, i // n_snap % n_ch
        stuck = q % 97 == 5
        cols = {"snap": s, "rank": rank[q], "comm": comm[q], "channel": ch, "seq_posted": np.where(stuck, 3, 4 + s),
                "chunks_sent": np.where(stuck, 2, s), "chunks_recv": np.where(stuck, 1, s)}
        cols = {k: v.astype(np.uint64 if k == "seq_posted" else np.uint32) for k, v in cols.items()}
        h, want = an.locate_hang(an.snapshots_to_device(cols), n_snap, n_ch), orc.Oracle(topo).locate_hang(cols, n_snap, n_ch)
        r, rate = an.progress_rates(an.snapshots_to_device(cols), n_snap, n_ch), orc.Oracle(topo).progress_rates(cols, n_snap, n_ch)
        assert h.status == want.status and r.status == rate.status, (n_snap, n_ch)
        assert all(np.array_equal(h.root[k], want.root[k]) for k in want.root), (n_snap, n_ch)
        assert all(np.array_equal(r.comm[k], rate.comm[k]) for k in rate.comm), (n_snap, n_ch)
    an.close()


@pytest.mark.parametrize("n_comms", [1, 510, 511, 512, 513, 1022, 1023, 1024, 1025, 1026])
def test_windows_around_the_rules_of_the_statistics(n_comms):
    """communicators of two and of 70 members, a fine bucket each: wavefronts per bucket, records summed or scanned"""
    topo = tg.make_topology(1024, [[c % 1000, c % 1000 + 1 + c // 1000] if c % 8 or n_comms > 600 else list(range(70)) for c in range(n_comms)])
    for rounds in (1, 3):
        m = [np.asarray(topo.members_of(c)) for c in range(n_comms)]
        comm = np.repeat(np.arange(n_comms), [x.size * rounds for x in m])
        rank = np.concatenate([np.tile(x, rounds) for x in m])
        seq = np.concatenate([np.repeat(np.arange(rounds), x.size) for x in m])
        rng = np.random.default_rng(n_comms)
        te = T0 + seq * 10**9 + rng.integers(0, 1000, comm.size)
        te[rng.random(comm.size) < 0.05] += 10**7
        keep = rng.random(comm.size) < 0.98
        keep[0] = True
        p = rng.permutation(np.flatnonzero(keep))
        cols = {"rank": rank.astype(np.uint32), "comm": comm.astype(np.uint32), "seq": seq.astype(np.uint64), "op": np.ones(comm.size, np.uint8),
                "bytes": np.full(comm.size, 64, np.uint64), "t_enter": te, "t_exit": te + 5 * 10**7}
        run_both(topo, {k: v[p] for k, v in cols.items()}, what=(n_comms, rounds))


@pytest.mark.parametrize("batches", [2, 5, 6, 11])
@pytest.mark.parametrize("n_comms", [1000, 1024, 1025, 2049, 3000])
def test_layout_of_several_batches(n_comms, batches):
    """counter ranges of more or fewer communicators than threads, of batches around the number that is loaded at a time; one is empty"""
    from paper_2605_04478_amd import ccld
    topo = tg.make_topology(1024, [[c % 1000, c % 1000 + 1 + c // 1000] for c in range(n_comms)])
    rng = np.random.default_rng(n_comms + batches)
    comm = np.tile(np.repeat(np.arange(n_comms), 2), 4)
    rank = np.tile(np.concatenate([topo.members_of(c) for c in range(n_comms)]), 4)
    seq = np.repeat(np.arange(4), 2 * n_comms) + 3 * comm
    te = T0 + (seq - 3 * comm) * 10**9 + rng.integers(0, 1000, comm.size)
    te[rng.random(comm.size) < 0.02] += 10**7
    p = rng.permutation(comm.size)
    cols = {"rank": rank.astype(np.uint32), "comm": comm.astype(np.uint32), "seq": seq.astype(np.uint64), "op": np.ones(comm.size, np.uint8),
            "bytes": np.full(comm.size, 64, np.uint64), "t_enter": te, "t_exit": te + 5 * 10**7}
    cols = {k: v[p] for k, v in cols.items()}
    cuts = np.sort(rng.integers(0, comm.size, batches - 2))
    cuts = np.concatenate([[0], cuts, cuts[-1:] if cuts.size else [0], [comm.size]])          # an empty batch before the last
    an = ccld.Analyzer(topo, max_window_records=comm.size, window_batches=batches)
    for lo, hi in zip(cuts[:-1], cuts[1:]):
        an.ingest(an.to_device({k: v[lo:hi] for k, v in cols.items()}))
    g = an.analyze_window(FAR, n_records=comm.size, per_record=True)
    compare(g, orc.Oracle(topo).analyze_window(cols, FAR), *an.rank_blame(), what=(n_comms, batches))
    an.close()
