"""GPU parity: ccld_flag_chains through the C ABI against the oracle's separation of root-cause and
secondary late entries (bit-exact tables), under both placements."""
import numpy as np
import pytest

from oracle import ccld_oracle as orc
from paper_2605_04478_amd import tracegen as tg
from tests.helpers import INFLIGHT, T0, toy_cols
from tests.test_oracle_chains import MS, _chain_case, _chain_case_without_gaps, _two_open_rows

pytestmark = pytest.mark.gpu


def run_both(topo, cols, now, what="", **params):
    from paper_2605_04478_amd import ccld
    o = orc.Oracle(topo, params)
    ref = o.analyze_window(cols, now)
    assert ref.status == "OK"
    chain, per_rank = o.flag_chains(cols, ref)
    n = int(cols["rank"].shape[0])
    for placement in (0, 1):
        an = ccld.Analyzer(topo, max_window_records=max(n, 1), placement=placement, **params)
        an.ingest(an.to_device(cols))
        g = an.analyze_window(now, n_records=n)
        st, gc, gr = an.flag_chains(g)
        assert st == "OK" and g.n_flag == len(ref.flag["comm"]), (what, st)
        for k in chain:
            assert np.array_equal(gc[k], chain[k]), (what, placement, k, np.nonzero(gc[k] != chain[k])[0][:5])
        for k in per_rank:
            assert np.array_equal(gr[k], per_rank[k]), (what, placement, k)
        # only the most recent analysis can be chained
        an.ingest(an.to_device({k: v[:0] for k, v in cols.items()}))
        with pytest.raises(ccld.CcldError):
            an.flag_chains(g)
        an.close()
    return chain, per_rank


def test_hand_built_chain_parity():
    topo, rows, _ = _chain_case()
    chain, per_rank = run_both(topo, toy_cols(rows), T0 + 10**12, what="chain")
    assert list(chain["depth"]) == [0, 1, 2, 1, 2] and list(per_rank["caused"])[0] == 5


def test_tie_rules_parity():
    for e0, e1 in ((T0, T0 + 100_000), (T0 + 100_000, T0), (T0, T0)):
        topo, rows = _two_open_rows(e0, e1)
        run_both(topo, toy_cols(rows), T0 + 10**12, what="two open operations")
    topo, rows = _chain_case_without_gaps()
    run_both(topo, toy_cols(rows), T0 + 10**12, what="no gaps")
    topo, rows, _ = _chain_case()
    rows = [(rk, c, s, op, nb, te, tx + (2 * MS if (rk, c, s) == (2, 0, 1) else 0)) for rk, c, s, op, nb, te, tx in rows]
    run_both(topo, toy_cols(rows), T0 + 10**12, what="late exit")


def test_truncated_collective_table_is_refused():
    from paper_2605_04478_amd import ccld
    topo, rows, _ = _chain_case()
    cols = toy_cols(rows)
    an = ccld.Analyzer(topo, max_window_records=len(rows))
    an.ingest(an.to_device(cols))
    g = an.analyze_window(T0 + 10**12, n_records=len(rows), seg_cap=2)
    assert g.status == "W_TRUNCATED" and g.n_seg == 4
    with pytest.raises(ccld.CcldError):
        an.flag_chains(g)
    g = an.analyze_window(T0 + 10**12, n_records=len(rows))
    st, chain, _ = an.flag_chains(g)
    assert st == "OK" and list(chain["depth"]) == [0, 1, 2, 1, 2]
    an.close()


def test_dependent_schedule_parity():
    spec = tg.config2(n_cycles=20)
    spec.same_size_per_kind = True
    tr = tg.propagate(tg.generate(spec), gap_ns=2_000_000).shuffled(3)
    chain, per_rank = run_both(tr.topo, tr.cols, int(tr.cols["t_exit"].max()) + 1, what="propagating")
    assert (chain["parent"] >= 0).sum() > 300 and chain["depth"].max() >= 2


def test_members_without_records_in_flight_operations_and_ties():
    """Rounds in which the flagged rank has no record, operations still in flight, equal exit times on two
    communicators, late exits, and a communicator of one member."""
    topo = tg.make_topology(9, [[0, 1, 2, 3], [0, 4, 5, 6], [0, 7], [8]])
    MS = 1_000_000
    rows = []

    def coll(comm, seq, enters, end=None, skip=()):
        end = max(enters.values()) + 400_000 if end is None else end
        for r, t in enters.items():
            if r not in skip:
                rows.append((r, comm, seq, tg.OP_ALLREDUCE, 1 << 20, t, end))
        return end
    t = T0
    for s in range(12):
        late1 = {1: 2 * MS} if s % 3 == 0 else {}
        e0 = coll(0, s, {r: t + late1.get(r, 0) for r in (0, 1, 2, 3)}, skip=(0,) if s in (4, 5) else ())
        # rank 0 goes on to communicator 1 (its peers there were ready long before), then to communicator 2
        e1 = coll(1, s, {0: e0 + 50_000, 4: t + 50_000, 5: t + 50_000, 6: t + 50_000})
        e2 = coll(2, s, {0: e1 + 50_000, 7: t + 50_000 + (3 * MS if s == 7 else 0)}, end=(e1 + 450_000 + (3 * MS if s == 7 else 0)))
        coll(3, s, {8: t})
        t = max(e2, t) + 5 * MS
    # the last round of communicator 1 never completes for two members
    rows = [(r, c, s, op, nb, te, (INFLIGHT if (c == 1 and s == 11 and r in (4, 5)) else tx)) for r, c, s, op, nb, te, tx in rows]
    cols = toy_cols(rows)
    p = np.random.default_rng(0).permutation(len(rows))
    run_both(topo, {k: v[p] for k, v in cols.items()}, t + 10**9, what="ragged")


def _jumps_in_step(parent):
    """Ancestors and links to them by doubling jumps of all flags at once: 2^i links after the i-th (a root stays)."""
    n = len(parent)
    anc = np.where(parent >= 0, parent, np.arange(n))
    depth = (parent >= 0).astype(np.int64)
    reach = 1
    while reach < n:
        nxt = anc[anc]
        depth = depth + np.where(nxt != anc, depth[anc], 0)
        anc, reach = nxt, 2 * reach
    return anc, depth


@pytest.mark.parametrize("loop,tail,sort", [(2, 0, False), (3, 1, False), (7, 40, True), (40, 3, False), (129, 200, True),
                                            (1500, 700, False)])
def test_clocks_that_contradict_each_other(loop, tail, sort):
    """Communicator i = {i, i + 1 modulo `loop`, two more}: its rank i enters late and its rank i + 1 has left before that,
    so the late entries name each other as parents all the way round; `tail` ranks whose chain leads into the loop, and one
    flag with a root.  Every flag then has the ancestor that jumps in step find, however often it is asked for."""
    from paper_2605_04478_amd import ccld
    LATE = 50 * MS
    comms, rows, r = [], [], loop + tail + 1

    def coll(members, late, t, seq=0):
        c = len(comms)
        comms.append(members)
        for m in members:
            te = t + (LATE if m == late else 0)
            rows.append((m, c, seq, tg.OP_ALLREDUCE, 1 << 20, te, te + MS // 2))

    for i in range(loop):
        coll(sorted({i, (i + 1) % loop}) + [r, r + 1, r + 2], i, T0)
        r += 3
    for j in range(tail):                   # rank loop + j: in the collective of the one before it, then late in its own
        coll([0 if j == 0 else loop + j - 1, loop + j, r, r + 1, r + 2], 0 if j == 0 else loop + j - 1, T0 + 10**10 + j * LATE * 3)
        r += 3
    coll([loop + tail, r, r + 1, r + 2], loop + tail, T0)
    r += 3
    if sort:                                # a round that nobody recorded: the window is sorted
        coll([r], -1, T0)
        rows.append((r, len(comms) - 1, 2, tg.OP_ALLREDUCE, 1 << 20, T0 + 10 * MS, T0 + 11 * MS))
        r += 1
    cols = toy_cols(rows)
    p = np.random.default_rng(loop).permutation(len(rows))
    cols = {k: v[p] for k, v in cols.items()}
    topo = tg.make_topology(r, comms)
    now = T0 + 10**13
    ref = orc.Oracle(topo).analyze_window(cols, now)
    n_flag, late = len(ref.flag["comm"]), ref.flag["rank"].astype(np.int64)
    assert n_flag == loop + tail + 1 and (ref.flag["kind"] & orc.FLAG_LATE_ENTER).all()
    with pytest.raises(ValueError):
        orc.Oracle(topo).flag_chains(cols, ref)              # it refuses loops
    parent = np.concatenate([(np.arange(loop) - 1) % loop, np.arange(loop - 1, loop + tail - 1), [-1]])
    if tail:                                # rank 0 leaves its late collective last, so its next one hangs on that
        parent[loop] = 0
    root, depth = _jumps_in_step(parent)
    per = {"root_entries": np.bincount(late[parent < 0], minlength=r), "secondary_entries": np.bincount(late[parent >= 0], minlength=r),
           "caused": np.bincount(late[root], minlength=r)}
    for placement in (0, 1):
        an = ccld.Analyzer(topo, max_window_records=len(rows), placement=placement)
        an.ingest(an.to_device(cols))
        g = an.analyze_window(now, n_records=len(rows))
        for again in range(4):
            st, chain, per_rank = an.flag_chains(g)
            assert st == "OK"
            for name, want in (("parent", parent), ("root", root), ("root_rank", late[root]), ("depth", depth)):
                assert np.array_equal(chain[name], want), (name, again, np.nonzero(chain[name] != want)[0][:5])
            for name in per:
                assert np.array_equal(per_rank[name], per[name]), (name, again)
        an.close()


@pytest.mark.parametrize("step", [1, 10**6], ids=["grid", "sorted"])
@pytest.mark.parametrize("rounds,many", [(900, False), (2300, True)])
def test_few_and_many_flags(rounds, many, step):
    """flags on both sides of the number from which fewer lanes search for a parent; ranks miss rounds and end in flight"""
    R = 64
    topo = tg.make_topology(R, [list(range(i, i + 8)) for i in range(0, R, 8)] + [list(range(i, R, 8)) for i in range(8)])
    rng = np.random.default_rng(rounds)
    q, half, rank = (x.reshape(-1) for x in np.meshgrid(np.arange(rounds), np.arange(2), np.arange(R), indexing="ij"))
    comm = np.where(half == 0, rank // 8, 8 + rank % 8)
    te = T0 + (2 * q + half) * 10 * MS + rng.integers(0, 1000, q.size)
    te[rng.random(q.size) < 0.1] += 3 * MS
    tx = T0 + (2 * q + half) * 10 * MS + 6 * MS + rng.integers(0, 1000, q.size)
    tx[(q == rounds - 1) & (half == 1) & (rng.random(q.size) < 0.3)] = INFLIGHT         # a rank's last operation
    keep = rng.random(q.size) < 0.99
    p = rng.permutation(np.flatnonzero(keep))
    cols = {"rank": rank.astype(np.uint32), "comm": comm.astype(np.uint32), "seq": (1 + q * step).astype(np.uint64), "op": np.ones(q.size, np.uint8),
            "bytes": np.full(q.size, 64, np.uint64), "t_enter": te, "t_exit": tx}
    chain, per_rank = run_both(topo, {k: v[p] for k, v in cols.items()}, int(T0 + rounds * 30 * MS), what=(rounds, step), hang_threshold_ns=10**15)
    assert (len(chain["parent"]) > 1 << 14) == many and (chain["parent"] >= 0).any()


@pytest.mark.parametrize("n,rounds,share", [(3, 30, 0.3), (16, 20, 0.2), (17, 20, 0.2), (63, 20, 0.1), (70, 20, 0.1), (1000, 12, 0.02), (4100, 8, 0.01),
                                            (4100, 45, 0.12)])
@pytest.mark.parametrize("step", [1, 10**6], ids=["grid", "sorted"])
def test_parents_among_many_late_members(n, rounds, share, step):
    """late members anywhere in collectives of fewer and of more members than lanes look for the parent, many with the same lag (the
    smallest rank is the parent); the last one is past the number of flags from which fewer lanes look"""
    topo = tg.make_topology(n, [list(range(n))])
    rng = np.random.default_rng(n + rounds)
    q, rank = np.repeat(np.arange(rounds), n), np.tile(np.arange(n), rounds)
    te = T0 + q * 10 * MS + np.where(rng.random(q.size) < share, rng.integers(2, 4, q.size) * MS, 0)
    p = rng.permutation(q.size)
    cols = {"rank": rank.astype(np.uint32), "comm": np.zeros(q.size, np.uint32), "seq": (1 + q * step).astype(np.uint64), "op": np.ones(q.size, np.uint8),
            "bytes": np.full(q.size, 64, np.uint64), "t_enter": te, "t_exit": T0 + q * 10 * MS + 6 * MS}
    chain, _ = run_both(topo, {k: v[p] for k, v in cols.items()}, int(T0 + rounds * 30 * MS), what=(n, step))
    assert (len(chain["parent"]) > 1 << 14) == (rounds == 45) and (chain["parent"] >= 0).any()
