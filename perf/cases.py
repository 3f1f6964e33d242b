"""The work that a user of the analyzer has it do, as cases that can be timed.

Every case drives the public Python entry points on inputs of its own: windows of trace records (ingest, analysis,
blame, flag chains), sliding windows fed batch by batch, hang location and progress rates on snapshot rows, and the
decoding of Probing Frames.  Inputs follow the distributions of `paper_2605_04478_amd.tracegen` (the same time model
and faults), drawn on the GPU so that large ones take a fraction of a second.

A case is a dict of plain values; "kind" names the path, the other fields are its sizes and options.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_04478_amd import ccld, tracegen as tg

DEV = "cuda:0"
EPOCH = tg.T_EPOCH_NS
HANG_THRESHOLD_NS = 5_000_000_000
OP_KINDS = ("tp", "pp", "dp", "world")
STREAM_PERIOD = 20                   # batches a stream keeps prepared (a multiple of the cycle's length)


def listed():
    return [
        # one ring of 16 ranks, 1,000 all-reduces: the smallest window, bound by launches and host waits
        window("window_16r", tp=16, pp=1, dp=1, slots=1000, cycle="ring"),
        # half a minute of a 512-rank job, with the separation of root cause and secondary late entries
        window("window_512r_chains", tp=8, pp=4, dp=16, slots=10_000, chains=True),
        # the 4,096-rank trace of the benchmark: 81.92M records in a random order
        window("window_4096r", tp=8, pp=8, dp=64, slots=20_000),
        # a quarter of that trace with the other placement
        window("window_4096r_dense", tp=8, pp=8, dp=64, slots=5_000, placement="dense"),
        # sizes that are no powers of two, records in time order, a world communicator, one hung operation, and
        # the per-record lags and order
        window("window_ragged", tp=6, pp=5, dp=13, slots=2_739, cycle="world", order="time", per_record=True, hung=True),
        # a batch that a collector hands over in ordinary host memory
        window("window_host", tp=8, pp=4, dp=16, slots=2_000, where="host"),
        # streaming at 16,384 ranks: 2M new records a second, window of ten batches
        stream("stream_16384r", tp=8, pp=16, dp=128, slots=122, batches=10),
        # streaming at 512 ranks: 62,464 new records a second
        stream("stream_512r", tp=8, pp=4, dp=16, slots=122, batches=10),
        # hang location on every (rank, communicator, channel) of 4,096 ranks over 64 snapshots
        snapshots("hang", "hang_4096r", tp=8, pp=8, dp=64, channels=16, snaps=64),
        # the same on a small job: 61,440 rows
        snapshots("hang", "hang_96r", tp=4, pp=3, dp=8, channels=4, snaps=40),
        # progress rates at a ragged size: 2.4M rows
        snapshots("rates", "rates_1008r", tp=8, pp=6, dp=21, channels=12, snaps=50),
        # one snapshot of 4,096 ranks as Probing Frames
        frames("frames_4096r", tp=8, pp=8, dp=64, channels=8),
    ]


def window(name=None, *, tp, pp, dp, slots, cycle="3d", order="shuffled", placement="sort", where="device",
           per_record=False, chains=False, hung=False):
    return _case(name, kind="window", tp=tp, pp=pp, dp=dp, slots=slots, cycle=cycle, order=order, placement=placement,
                 where=where, per_record=per_record, chains=chains, hung=hung)


def stream(name=None, *, tp, pp, dp, slots, batches, order="time"):
    return _case(name, kind="stream", tp=tp, pp=pp, dp=dp, slots=slots, batches=batches, order=order)


def snapshots(kind, name=None, *, tp, pp, dp, channels, snaps, healthy=False, where="device", static=False):
    return _case(name, kind=kind, tp=tp, pp=pp, dp=dp, channels=channels, snaps=snaps, healthy=healthy, where=where,
                 static=static)


def frames(name=None, *, tp, pp, dp, channels, where="device"):
    return _case(name, kind="frames", tp=tp, pp=pp, dp=dp, channels=channels, where=where)


def _case(name, **fields):
    return fields if name is None else dict(name=name, **fields)


# ---- further cases of the same ranges --------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _layout(rng, max_ranks):
    """A parallel layout as jobs have it: a node-sized tensor group, some pipeline stages, the rest data parallel."""
    while True:
        tp, pp, dp = rng.choice((2, 3, 4, 5, 6, 7, 8, 8, 8, 12, 16)), _log_int(rng, 2, 16), _log_int(rng, 2, 128)
        if tp * pp * dp <= max_ranks:
            return dict(tp=tp, pp=pp, dp=dp)


def draw(rng):
    kind = rng.choices(("window", "stream", "hang", "rates", "frames"), (5, 2, 2, 1, 1))[0]
    if kind == "window":
        lay = _layout(rng, 4096)
        ranks = lay["tp"] * lay["pp"] * lay["dp"]
        slots = max(11, _log_int(rng, 1_000, 40_000_000) // ranks)
        n = slots * ranks
        return window(**lay, slots=slots, cycle="world" if rng.random() < 0.3 else "3d",
                      order=rng.choice(("shuffled", "time")), placement="dense" if rng.random() < 0.25 else "sort",
                      where="host" if n <= 2_000_000 and rng.random() < 0.25 else "device",
                      per_record=n <= 4_000_000 and rng.random() < 0.2, chains=rng.random() < 0.3,
                      hung=rng.random() < 0.3)
    if kind == "stream":
        lay = _layout(rng, 16384)
        ranks = lay["tp"] * lay["pp"] * lay["dp"]
        batches = rng.randint(4, 16)
        slots = max(2, min(400, _log_int(rng, 2_000, 20_000_000) // (ranks * batches)))
        return stream(**lay, slots=slots, batches=batches, order=rng.choice(("shuffled", "time")))
    lay = _layout(rng, 4096)
    members = 4 * lay["tp"] * lay["pp"] * lay["dp"]
    if kind == "frames":
        return frames(**lay, channels=rng.randint(1, 8), where=rng.choice(("device", "host")))
    snaps = _log_int(rng, 32, 128)
    channels = max(1, min(16, _log_int(rng, 4_000, 16_000_000) // (members * snaps)))
    rows = members * channels * snaps
    small = kind == "hang" and rows <= 400_000 and members <= 8_000
    return snapshots(kind, **lay, channels=channels, snaps=snaps, healthy=rng.random() < 0.25,
                     where="host" if rows <= 1_000_000 and rng.random() < 0.25 else "device",
                     static=small and rng.random() < 0.3)


# ---- what the path cannot do without -----------------------------------------------------------------------
def _cycle(case):
    if case.get("cycle") == "ring":
        return (("tp", tg.OP_ALLREDUCE),)
    return tg.CYCLE_3D + (tg.CYCLE_WORLD if case.get("cycle") == "world" else ())


def _comms_of_kind(lay, kind):
    return {"tp": lay.n_tp, "pp": lay.n_pp, "dp": lay.n_dp, "world": 1}[kind]


def _collectives(case, lay):
    cyc = _cycle(case)
    per = [_comms_of_kind(lay, k) for k, _ in cyc]
    return case["slots"] // len(cyc) * sum(per) + sum(per[:case["slots"] % len(cyc)])


def work(case):
    lay = _lay(case)
    ranks, members = lay.n_ranks, 4 * lay.n_ranks
    if case["kind"] == "window":
        # the 41-byte records in; the 21-column collective table, the blame table and its order, and the
        # per-record outputs where they are wanted, out
        n = case["slots"] * ranks
        return {"bytes": 41 * n + 168 * _collectives(case, lay) + 44 * ranks + (21 * n if case["per_record"] else 0),
                "flops": 0}
    if case["kind"] == "stream":
        # the new records in, the table of the whole window out
        n = case["slots"] * ranks
        return {"bytes": 41 * n + 168 * case["batches"] * _collectives(case, lay) + 44 * ranks, "flops": 0}
    if case["kind"] == "frames":
        return {"bytes": (tg.FRAME_BYTES + 4) * ranks + 32 * members * case["channels"], "flops": 0}
    comms = sum(_comms_of_kind(lay, k) for k in OP_KINDS)
    rows = members * case["channels"] * case["snaps"]
    per_member, per_comm = (80, 48) if case["kind"] == "hang" else (48, 32)
    return {"bytes": 32 * rows + per_member * members + per_comm * comms, "flops": 0}


def tolerance(case):
    return "exact"                   # every output is a whole number


# ---- trace records -----------------------------------------------------------------------------------------
def _lay(case):
    world = case["kind"] in ("hang", "rates", "frames") or case.get("cycle") == "world"
    return tg.Layout3D(tp=case["tp"], pp=case["pp"], dp=case["dp"], world=world)


class _Source:
    """Slot-major records of one simulated job: constant clock skews, a few slow ranks and one node with a slow link."""

    def __init__(self, lay, cycle, gen, slot_ns, size_exp, sigma=0.2, skew_ns=100_000):
        self.lay, self.cycle, self.gen, self.slot_ns, self.size_exp, self.sigma = lay, cycle, gen, slot_ns, size_exp, sigma
        R = lay.n_ranks
        self.skew = torch.randint(-skew_ns, skew_ns + 1, (R,), generator=gen, device=DEV)
        # large jobs: one rank in 512 is late on every operation; small ones: one rank on a tenth of them
        self.slow = torch.randperm(R, generator=gen, device=DEV)[:max(1, R // 512)]
        self.slow_prob = 1.0 if R >= 512 else 0.1
        node = int(torch.randint(0, R // lay.tp, (1,), generator=gen, device=DEV))
        self.stretch = torch.ones(R, dtype=torch.float64, device=DEV)
        self.stretch[node * lay.tp:(node + 1) * lay.tp] = 1.3

    def _rand(self, *shape):
        return torch.rand(shape, generator=self.gen, device=DEV, dtype=torch.float64)

    def slots(self, k0, k1):
        lay, cyc, R, S = self.lay, self.cycle, self.lay.n_ranks, k1 - k0
        i64 = dict(dtype=torch.int64, device=DEV)
        out = {"rank": torch.arange(R, dtype=torch.int32, device=DEV).repeat(S, 1),
               "comm": torch.empty((S, R), dtype=torch.int32, device=DEV), "seq": torch.empty((S, R), **i64),
               "op": torch.empty((S, R), dtype=torch.uint8, device=DEV), "bytes": torch.empty((S, R), **i64),
               "t_enter": torch.empty((S, R), **i64), "t_exit": torch.empty((S, R), **i64)}
        ks_all = np.arange(k0, k1)
        for kind in dict(cyc):
            pos = [i for i, (kd, _) in enumerate(cyc) if kd == kind]
            ks = ks_all[np.isin(ks_all % len(cyc), pos)]
            if not ks.size:
                continue
            m = ks.size
            comm = torch.from_numpy(np.asarray(lay.comm_of(kind, np.arange(R)), dtype=np.int64)).to(DEV)
            group = comm - comm.min()
            n_groups = _comms_of_kind(lay, kind)
            ordinal = np.searchsorted(pos, ks % len(cyc))
            seq = torch.from_numpy(ks // len(cyc) * len(pos) + ordinal).to(DEV)
            ops = torch.from_numpy(np.asarray([cyc[p][1] for p in ks % len(cyc)], dtype=np.uint8)).to(DEV)
            lo, hi = self.size_exp
            nbytes = torch.floor(torch.exp2(lo + (hi - lo) * self._rand(m, n_groups)))
            jitter = torch.exp(self.sigma * torch.randn((m, n_groups), generator=self.gen, device=DEV, dtype=torch.float64))
            enter = torch.floor(self._rand(m, R) * 20_000)
            late = torch.floor(-1_000_000 * torch.log1p(-self._rand(m, self.slow.numel()))).clamp_(min=1)
            late *= self._rand(m, self.slow.numel()) < self.slow_prob
            enter[:, self.slow] += late
            enter += torch.from_numpy(ks.astype(np.float64) * self.slot_ns).to(DEV)[:, None]
            dims = {"tp": (3,), "pp": (1,), "dp": (2,), "world": (1, 2, 3)}[kind]
            e4 = enter.view(m, lay.pp, lay.dp, lay.tp)
            exit_ = e4.amax(dim=dims, keepdim=True).expand_as(e4).reshape(m, R)
            dur = (nbytes / 20.0 * jitter)[:, group]
            if kind == "dp":
                dur = dur * self.stretch
            exit_ = exit_ + torch.round(dur) + torch.floor(self._rand(m, R) * 5_000)
            rows = torch.from_numpy(ks - k0).to(DEV)
            out["comm"][rows] = comm.to(torch.int32)
            out["seq"][rows] = seq[:, None].expand(m, R)
            out["op"][rows] = ops[:, None].expand(m, R)
            out["bytes"][rows] = nbytes.to(torch.int64)[:, group]
            out["t_enter"][rows] = EPOCH + enter.to(torch.int64) + self.skew
            out["t_exit"][rows] = EPOCH + exit_.to(torch.int64) + self.skew
        return {k: v.view(-1) for k, v in out.items()}


def _shuffle(cols, gen):
    perm = torch.randperm(cols["rank"].numel(), generator=gen, device=DEV)
    return {k: v[perm] for k, v in cols.items()}


_HOST_DTYPES = {"rank": np.uint32, "comm": np.uint32, "seq": np.uint64, "op": np.uint8, "bytes": np.uint64,
                "t_enter": np.int64, "t_exit": np.int64, "snap": np.uint32, "channel": np.uint32,
                "seq_posted": np.uint64, "chunks_sent": np.uint32, "chunks_recv": np.uint32}


def _to_host(cols):
    return {k: v.cpu().numpy().view(_HOST_DTYPES[k]) for k, v in cols.items()}


def _result_buffers(an, n, n_seg, per_record):
    """Result tables that serve every pass (rows past a table's count keep what they held)."""
    buffers = an.alloc_window_result(n, seg_cap=n_seg, flag_cap=n // 12 + 1024, group_cap=min(n_seg, an.n_comms * 1024),
                                     alert_cap=1024, cand_cap=16384, per_record=per_record)
    for t in buffers[1].values():
        t.zero_()
    blame = (torch.empty(len(ccld.BLAME_COLS) * an.n_ranks, dtype=torch.int64, device=DEV),
             torch.empty(an.n_ranks, dtype=torch.int32, device=DEV))
    return buffers, blame


def _window_outputs(s, res):
    counts = [res.n_records, res.n_seg, res.n_flag, res.n_group, res.n_alert, res.n_cand]
    return {"ok": res.status == "OK", "counts": counts, "tables": s["buffers"][1], "blame": s["blame"]}


def _prepare_window(case, gen):
    lay, cyc = _lay(case), _cycle(case)
    size_exp = (20.0, 28.0) if lay.n_ranks <= 512 else (16.0, 29.0)
    slot_ns = 100_000_000 if lay.n_ranks <= 512 else 250_000_000
    cols = _Source(lay, cyc, gen, slot_ns, size_exp).slots(0, case["slots"])
    if case["hung"]:
        # one member of the first data-parallel communicator does not enter its last operation; the peers wait in it
        comm = int(lay.comm_of("dp", np.zeros(1, dtype=np.int64))[0])
        on = cols["comm"] == comm
        last = on & (cols["seq"] == cols["seq"][on].max())
        cols["t_exit"][last] = tg.INFLIGHT
        cols = {k: v[~(last & (cols["rank"] == 0))] for k, v in cols.items()}
    if case["order"] == "shuffled":
        cols = _shuffle(cols, gen)
    n = cols["rank"].numel()
    placement = ccld.PLACEMENT_DENSE if case["placement"] == "dense" else ccld.PLACEMENT_SORT
    an = ccld.Analyzer(lay.topology(), max_window_records=n, device=DEV, placement=placement,
                       hang_threshold_ns=HANG_THRESHOLD_NS)
    buffers, blame = _result_buffers(an, n, _collectives(case, lay), case["per_record"])
    # successive windows of the job: the operation counters go on, the other columns serve again
    windows = []
    for i in range(4):
        w = dict(cols, seq=cols["seq"] + i * case["slots"])
        windows.append(_to_host(w) if case["where"] == "host" else w)
    s = {"kind": "window", "an": an, "windows": windows, "at": 0, "buffers": buffers, "blame": blame,
         "now": EPOCH + case["slots"] * slot_ns + 2 * HANG_THRESHOLD_NS}
    if case["chains"]:               # the report that the chains are collected in
        s["chains"] = np.zeros((len(ccld.CHAIN_COLS), buffers[0]["flag"]), dtype=np.int64)
    return s


def _run_window(s):
    an, w = s["an"], s["windows"][s["at"] % len(s["windows"])]
    s["at"] += 1
    an.reset_window()
    an.ingest(w)
    res = an.analyze_window(s["now"], buffers=s["buffers"])
    an.rank_blame(to_host=False, buffers=s["blame"])
    out = _window_outputs(s, res)
    if "chains" in s:
        status, chain, per_rank = an.flag_chains(res)
        for i, name in enumerate(ccld.CHAIN_COLS):
            s["chains"][i, :res.n_flag] = chain[name]
        out["chains"] = {"ok": status == "OK", "per_flag": s["chains"], "per_rank": per_rank}
    return out


def _prepare_stream(case, gen):
    lay, cyc, slots, W = _lay(case), _cycle(case), case["slots"], case["batches"]
    source = _Source(lay, cyc, gen, 8_192_000, (16.0, 25.0))
    batches = []
    for b in range(STREAM_PERIOD):
        cols = source.slots(b * slots, (b + 1) * slots)
        batches.append(_shuffle(cols, gen) if case["order"] == "shuffled" else cols)
    per = slots * lay.n_ranks
    an = ccld.Analyzer(lay.topology(), max_window_records=W * per, max_batch_records=per, window_batches=W,
                       hang_threshold_ns=HANG_THRESHOLD_NS, device=DEV)
    buffers, blame = _result_buffers(an, W * per, W * (_collectives(case, lay) + 2 * an.n_comms), False)
    # what a communicator's operation counter advances by until a prepared batch comes round again
    per_cycle = {k: sum(kd == k for kd, _ in cyc) for k in dict(cyc)}
    advance = torch.cat([torch.full((_comms_of_kind(lay, k),), STREAM_PERIOD * slots // len(cyc) * per_cycle[k])
                         for k in ("tp", "pp", "dp")]).to(DEV)
    s = {"kind": "stream", "an": an, "batches": batches, "advance": [advance[b["comm"].long()] for b in batches],
         "period_ns": STREAM_PERIOD * slots * 8_192_000, "batch_ns": slots * 8_192_000, "step": 0,
         "buffers": buffers, "blame": blame}
    for _ in range(W):                # the job has been watched for a window's length
        _run_stream(s)
    return s


def _run_stream(s):
    an, i = s["an"], s["step"]
    b, advance = s["batches"][i % STREAM_PERIOD], s["advance"][i % STREAM_PERIOD]
    if i >= STREAM_PERIOD:            # the next seconds of the job: later counters and times
        b["seq"].add_(advance)
        torch._foreach_add_([b["t_enter"], b["t_exit"]], s["period_ns"])
    s["step"] = i + 1
    an.ingest(b)
    res = an.analyze_window(EPOCH + (i + 1) * s["batch_ns"], buffers=s["buffers"])
    an.rank_blame(to_host=False, buffers=s["blame"])
    return _window_outputs(s, res)


# ---- snapshots ---------------------------------------------------------------------------------------------
def _snapshot_rows(lay, snaps, channels, per_kind, gen):
    """Columns of every (snapshot, rank, communicator, channel) in a random order; per_kind(kind, group, n_groups) gives
    the operation counter and the two counts as [snapshots, ranks, channels] (or what broadcasts to it)."""
    R = lay.n_ranks
    shape = (snaps, R, channels)
    parts = {k: [] for k in tg.SNAP_COLUMNS}
    i32 = lambda t: t.to(torch.int32).expand(shape).reshape(-1)
    for kind in OP_KINDS:
        comm = torch.from_numpy(np.asarray(lay.comm_of(kind, np.arange(R)), dtype=np.int64)).to(DEV)
        seq, sent, recv = per_kind(kind, comm - comm.min(), _comms_of_kind(lay, kind))
        parts["snap"].append(i32(torch.arange(snaps, device=DEV)[:, None, None]))
        parts["rank"].append(i32(torch.arange(R, device=DEV)[None, :, None]))
        parts["comm"].append(i32(comm[None, :, None]))
        parts["channel"].append(i32(torch.arange(channels, device=DEV)[None, None, :]))
        parts["seq_posted"].append(seq.to(torch.int64).expand(shape).reshape(-1))
        parts["chunks_sent"].append(i32(sent))
        parts["chunks_recv"].append(i32(recv))
    return _shuffle({k: torch.cat(v) for k, v in parts.items()}, gen)


def _hang_rows(case, lay, gen):
    """Completed operations everywhere until one rank of one data-parallel ring freezes; its ring runs until blocked,
    every other rank posts one more operation where a member of the ring is awaited."""
    R, snaps, ch = lay.n_ranks, case["snaps"], case["channels"]
    at = snaps + 1 if case["healthy"] else max(1, snaps // 4)
    root = int(torch.randint(0, R, (1,), generator=gen, device=DEV))
    ring_comm = int(lay.comm_of("dp", np.asarray([root]))[0])
    ring = np.nonzero(np.asarray(lay.comm_of("dp", np.arange(R))) == ring_comm)[0]
    c0 = torch.randint(100, 1000, (ch,), generator=gen, device=DEV).cpu().numpy()
    S, Rv = tg.ring_steady_state(len(ring), int(np.nonzero(ring == root)[0][0]), c0, 1 << 20, 8)
    ring = torch.from_numpy(ring).to(DEV)
    S, Rv = torch.from_numpy(S).to(DEV), torch.from_numpy(Rv).to(DEV)
    in_ring = torch.zeros(R, dtype=torch.bool, device=DEV)
    in_ring[ring] = True
    s_eff = torch.arange(snaps, device=DEV).clamp(max=at - 1)

    def per_kind(kind, group, n_groups):
        pace = torch.randint(1, 6, (n_groups,), generator=gen, device=DEV)
        base = torch.randint(1000, 10_000, (n_groups,), generator=gen, device=DEV)
        total = torch.randint(64, 2048, (n_groups, snaps, ch), generator=gen, device=DEV)
        seq = (base + pace * s_eff[:, None])[:, group][:, :, None].expand(snaps, R, ch).contiguous()
        sent = total[:, s_eff].transpose(0, 1)[:, group].contiguous()
        recv = sent.clone()
        if at < snaps:
            if kind == "dp":
                seq[at:, ring] = 12_345
                sent[at:, ring], recv[at:, ring] = S, Rv
            else:
                touched = torch.zeros(n_groups, dtype=torch.bool, device=DEV)
                touched[group[ring]] = True
                blocked = (touched[group] & ~in_ring).nonzero().view(-1)
                seq[at:, blocked] += 1
                sent[at:, blocked], recv[at:, blocked] = 1, 0
        return seq, sent, recv
    return _snapshot_rows(lay, snaps, ch, per_kind, gen)


def _rate_rows(case, lay, gen):
    """Operations of 8 chunks back to back every 10 samples; a healthy rank's count moves at 1 to 3 samples of an
    operation, the slow rank's at 6 to 8."""
    R, snaps, ch = lay.n_ranks, case["snaps"], case["channels"]
    slow = int(torch.randint(0, R, (1,), generator=gen, device=DEV))
    n_ops = snaps // 10 + 2

    def per_kind(kind, group, n_groups):
        phase = torch.randint(0, 10, (n_groups,), generator=gen, device=DEV)[group]
        first = torch.randint(1000, 10_000, (n_groups,), generator=gen, device=DEV)[group]
        since = torch.arange(snaps, device=DEV)[:, None] - phase                        # [snapshots, ranks]
        op = torch.div(since, 10, rounding_mode="floor")
        at = (op + 1)[:, :, None].expand(snaps, R, ch)
        done, counts = (since - 10 * op)[:, :, None], []
        for _ in range(2):
            k = torch.randint(1, 4, (n_ops, R, ch), generator=gen, device=DEV)
            if not case["healthy"]:
                k[:, slow] += 5
            k = torch.gather(k, 0, at)
            counts.append(torch.where(op[:, :, None] < 0, 8, 8 * torch.minimum(done, k) // k))
        return (first + op)[:, :, None], counts[0], counts[1]
    return _snapshot_rows(lay, snaps, ch, per_kind, gen)


def _prepare_snapshots(case, gen):
    lay = _lay(case)
    cols = (_hang_rows if case["kind"] == "hang" else _rate_rows)(case, lay, gen)
    an = ccld.Analyzer(lay.topology(), max_window_records=1024, max_snapshot_rows=cols["snap"].numel(), device=DEV)
    s = {"kind": case["kind"], "an": an, "cols": _to_host(cols) if case["where"] == "host" else cols,
         "snaps": case["snaps"], "channels": case["channels"], "static": case["static"]}
    if case["kind"] == "hang":
        caps = {"root": 4096, "pair": 4 * lay.n_ranks, "comm": an.n_comms}
        names = {"root": ccld.HANG_ROOT_COLS, "pair": ccld.HANG_PAIR_COLS, "comm": ccld.HANG_COMM_COLS}
        s["buffers"] = caps, {k: torch.zeros(len(v) * caps[k], dtype=torch.int64, device=DEV) for k, v in names.items()}
    return s


def _run_hang(s):
    res = s["an"].locate_hang(s["cols"], s["snaps"], s["channels"], static=s["static"], buffers=s["buffers"])
    return {"ok": res.status == "OK", "counts": [res.n_root, res.n_hung_comm], "tables": res.dev}


def _run_rates(s):
    res = s["an"].progress_rates(s["cols"], s["snaps"], s["channels"])
    return {"ok": res.status == "OK", "tables": res.dev}


# ---- Probing Frames ----------------------------------------------------------------------------------------
FRAME_SETS = 4                       # snapshots that are kept prepared


def _prepare_frames(case, gen):
    """One frame per rank: its communicators in consecutive blocks, which move on from snapshot to snapshot; a tenth of
    the communicators has left its rank's frame."""
    lay, ch = _lay(case), case["channels"]
    R, rng = lay.n_ranks, np.random.default_rng(int(torch.randint(0, 1 << 30, (1,), generator=gen, device=DEV)))
    sets = []
    for i in range(FRAME_SETS):
        f = np.zeros(R, dtype=tg.FRAME_DTYPE)
        f["mode"], f["n_channels"], f["counter"], f["kernel_index"] = 1, ch, 3 * i + 7, (3 * i + 7) % tg.FRAME_BLOCKS
        for k, kind in enumerate(OP_KINDS):
            comm = np.asarray(lay.comm_of(kind, np.arange(R)))
            b = (3 * i + k) % tg.FRAME_BLOCKS
            f["block"]["comm"][:, b] = comm
            f["block"]["ext"][:, b] = rng.random(R) >= 0.1
            f["block"]["counter"][:, b] = 1000 + 17 * comm + i
            f["block"]["count"][:, b, :ch] = rng.integers(0, 2048, (R, ch, 2))
        ranks = rng.permutation(R).astype(np.uint32)
        raw = f[ranks].view(np.uint8).reshape(-1)
        if case["where"] == "device":
            sets.append((torch.from_numpy(raw).to(DEV), torch.from_numpy(ranks.view(np.int32)).to(DEV)))
        else:
            sets.append((raw, ranks))
    # the operation counters of all eight blocks, which advance from one snapshot to the next
    words = [x[0].view(torch.int64 if case["where"] == "device" else np.int64).reshape(R, tg.FRAME_BYTES // 8)
             for x in sets]
    an = ccld.Analyzer(lay.topology(), max_window_records=1024, max_snapshot_rows=max(64 * R, 4 * R * ch), device=DEV)
    return {"kind": "frames", "an": an, "sets": sets, "counters": [w[:, 5::18] for w in words], "channels": ch, "snap": 0}


def _run_frames(s):
    i = s["snap"]
    frames_, ranks = s["sets"][i % FRAME_SETS]
    if i >= FRAME_SETS:
        counters = s["counters"][i % FRAME_SETS]
        counters += FRAME_SETS
    s["snap"] = i + 1
    status, rows = s["an"].decode_frames(frames_, ranks, i, s["channels"])
    return {"ok": status == "OK", "rows": rows}


# ---- entry points ------------------------------------------------------------------------------------------
_PREPARE = {"window": _prepare_window, "stream": _prepare_stream, "hang": _prepare_snapshots, "rates": _prepare_snapshots,
            "frames": _prepare_frames}
_RUN = {"window": _run_window, "stream": _run_stream, "hang": _run_hang, "rates": _run_rates, "frames": _run_frames}


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return _PREPARE[case["kind"]](case, gen)


def run(state):
    return _RUN[state["kind"]](state)
