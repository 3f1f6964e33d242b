"""GPU parity for streaming analysis: a sliding window of one-second batches kept on the device,
a slow rank that rotates, and a hang that appears mid-stream; every step is compared with the
CPU oracle run on the concatenated window."""
import numpy as np
import pytest

from oracle import ccld_oracle as orc
from paper_2605_04478_amd import tracegen as tg
from tests.test_gpu_window import compare

pytestmark = pytest.mark.gpu


def test_streaming_window_matches_oracle_every_step():
    from paper_2605_04478_amd import ccld
    ss = tg.config5(n_steps=26, layout=tg.Layout3D(tp=4, pp=4, dp=16), epoch_steps=6, hang_step=11)
    topo = ss.layout.topology()
    W = 10
    per = ss.slots_per_step * ss.layout.n_ranks
    params = dict(hang_threshold_ns=5_000_000_000, window_batches=W)
    an = ccld.Analyzer(topo, max_window_records=W * per, max_batch_records=per, **params)
    o = orc.Oracle(topo, dict(hang_threshold_ns=5_000_000_000))
    batches = []
    alerts_seen, located = [], set()
    hang_rank, hang_comm, hang_seq = ss.hang_site()
    for step in range(ss.n_steps):
        b = tg.stream_batch(ss, step)
        batches.append(b.cols)
        an.ingest(an.to_device(b.cols))
        win = batches[max(0, step - W + 1): step + 1]
        cols = {k: np.concatenate([w[k] for w in win]) for k in b.cols}
        now = ss.now_ns(step)
        g = an.analyze_window(now, n_records=W * per, per_record=True)
        ref = o.analyze_window(cols, now)
        blame, order = an.rank_blame()
        compare(g, ref, blame, order, what=f"step{step}")
        if g.n_alert:
            alerts_seen.append(step)
            a = g.alert
            assert list(a["comm"]) == [hang_comm] and list(a["seq"]) == [hang_seq] and list(a["class"]) == [1]
            assert list(g.cand) == [hang_rank]
        # the slow rank of the current epoch leads the blame once its epoch fills most of the window
        if step % ss.epoch_steps == ss.epoch_steps - 1:
            located.add((int(order[0]), ss.slow_rank(step)))
    # the hang is in flight for longer than 5 s from step hang+5 until its records leave the window
    assert alerts_seen == list(range(ss.hang_step + 5, ss.hang_step + W))
    assert all(a == b for a, b in located) and len(located) >= 3


def test_kept_window_order_survives_odd_sequences():
    """Windows of several batches that are placed on the grid, which keep nothing from one analysis to the next but the
    detection state.  The sequence of calls varies: several ingests between two analyses, an empty batch, batches
    of very different sizes, a hang location in between (it borrows the sort buffers), a reset, and
    operation counters that move the grid from step to step.  (The next test has windows that are sorted, whose order is
    kept.)"""
    from paper_2605_04478_amd import ccld
    from tests.test_gpu_window import FAR
    from tests.test_oracle_hang import snap_rows
    spec = tg.config2(n_cycles=40)
    tr = tg.generate(spec)
    R = spec.layout.n_ranks
    sizes = [7, 1, 0, 12, 3, 3, 25, 2, 9, 9, 4, 30, 1, 1, 6]           # collectives per rank in each batch
    starts = np.cumsum([0] + sizes)
    batches = [{k: v[starts[i] * R:starts[i + 1] * R] for k, v in tr.cols.items()} for i in range(len(sizes))]
    wb = 4
    cap = max(sum(sizes[i:i + wb]) for i in range(len(sizes))) * R + 13
    n_cells = int(tr.topo.size.sum()) * 4
    an = ccld.Analyzer(tr.topo, max_window_records=cap, max_batch_records=max(sizes) * R, window_batches=wb,
                       max_snapshot_rows=n_cells, stall_snapshots=2)
    o = orc.Oracle(tr.topo, dict(window_batches=wb, stall_snapshots=2))
    rng = np.random.default_rng(5)
    held = []
    for i, b in enumerate(batches):
        p = rng.permutation(len(b["rank"]))
        b = {k: v[p] for k, v in b.items()}
        if i == 11:                                          # start over: the kept order must not be used
            an.reset_window()
            held = []
        an.ingest(an.to_device(b))
        held = (held + [b])[-wb:]
        if i in (1, 5, 9):                                   # no analysis after these ingests
            continue
        if i == 7:                                           # the hang pass sorts its roots in the same buffers
            rows = snap_rows(tr.topo, 4, 1, lambda s, c, q, ch: (3, 5, 5) if q else (2, 9, 9))
            h = an.locate_hang(an.snapshots_to_device(rows), 4, 1, root_cap=n_cells)
            assert h.status == "OK" and h.n_root > 0
        cols = {k: np.concatenate([w[k] for w in held]) for k in b}
        n = len(cols["rank"])
        g = an.analyze_window(FAR, n_records=max(n, 1), per_record=True)
        ref = o.analyze_window(cols, FAR)
        blame, order = an.rank_blame()
        compare(g, ref, blame, order, what=f"batch{i}")
    an.close()


@pytest.mark.parametrize("wb,sizes", [(4, [7, 1, 0, 12, 3, 3, 25, 2, 9, 9, 4, 30, 1, 1, 6]), (2, [5, 5, 1, 6, 2]),
                                      (3, [40, 20, 21, 19, 1, 0, 0, 1, 50, 2])])
def test_kept_order_of_windows_that_are_sorted(wb, sizes):
    """The same with windows that cannot be placed on a grid (one communicator has 2,100 members): the kept order, merged with
    the new records, must be the one that sorting the window gives, whatever the sequence of calls; a batch with a
    duplicate fails and leaves no order behind."""
    from paper_2605_04478_amd import ccld
    from tests.helpers import T0, concat_cols, toy_cols
    from tests.test_gpu_window import FAR
    from tests.test_oracle_hang import snap_rows
    R = 2100
    comms = [list(range(R))] + [[4 * c + i for i in range(4)] for c in range(60)] + [[5]]
    topo = tg.make_topology(R, comms)
    rng = np.random.default_rng(wb)

    def batch(i):                                            # some communicators' counters run ahead, some stand still
        rows = []
        for j in range(starts[i], starts[i + 1]):
            for c, mem in enumerate(comms):
                if (c == 0 and j % 9) or (c and rng.random() < 0.1):
                    continue
                late = mem[int(rng.integers(0, len(mem)))]
                for r in mem:
                    te = T0 + j * 10**8 + int(rng.integers(0, 2000)) + (10**7 if r == late and j % 4 == 0 else 0)
                    rows.append((r, c, (1 << 33) + j * (1 + 300 * (c == 7)), 0, 1 << 20, te, te + 10**6 + int(rng.integers(0, 3000))))
        p = rng.permutation(len(rows))
        return {k: v[p] for k, v in toy_cols(rows).items()}

    starts = np.cumsum([0] + sizes)
    batches = [batch(i) for i in range(len(sizes))]
    n_b = [len(b["rank"]) for b in batches]
    cap = max(sum(n_b[i:i + wb]) for i in range(len(n_b))) + 13
    n_cells = int(topo.size.sum()) * 4
    an = ccld.Analyzer(topo, max_window_records=cap, max_batch_records=max(n_b) + 1, window_batches=wb, max_snapshot_rows=n_cells, stall_snapshots=2)
    o = orc.Oracle(topo, dict(window_batches=wb, stall_snapshots=2))
    held = []
    for i, b in enumerate(batches):
        if i == 11:
            an.reset_window()
            held = []
        if i == 4:                                           # a duplicate: an error, and the batch has to leave first
            an.reset_window()
            an.ingest(an.to_device(concat_cols(b, {k: v[:1] for k, v in b.items()})))
            assert an.analyze_window(FAR, n_records=cap, seg_cap=cap).status == ("E_DUPLICATE_KEY" if len(b["rank"]) else "OK")
            an.reset_window()
            held = []
        an.ingest(an.to_device(b))
        held = (held + [b])[-wb:]
        if i in (1, 9):                                      # no analysis after these ingests
            continue
        if i == 7:                                           # the hang pass sorts its roots in the same buffers
            rows = snap_rows(topo, 4, 1, lambda s, c, q, ch: (3, 5, 5) if q else (2, 9, 9))
            h = an.locate_hang(an.snapshots_to_device(rows), 4, 1, root_cap=n_cells)
            assert h.status == "OK" and h.n_root > 0
        cols = {k: np.concatenate([w[k] for w in held]) for k in b}
        n = len(cols["rank"])
        g = an.analyze_window(FAR, n_records=max(n, 1), per_record=True)
        ref = o.analyze_window(cols, FAR)
        compare(g, ref, *an.rank_blame(), what=f"batch{i}")
        if g.n_flag:
            st, chain, per_rank = an.flag_chains(g)
            assert st == "OK" and len(chain["parent"]) == g.n_flag
    an.close()
