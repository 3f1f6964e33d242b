"""GPU parity of the blame sums and the blame order at the edges of their kernels: more flagged ranks than a
workgroup's LDS table holds, and numbers of ranks around the tiles and the limit of the one-launch order."""
import numpy as np
import pytest

from oracle import ccld_oracle as orc
from paper_2605_04478_amd import tracegen as tg
from tests.helpers import T0, toy_cols
from tests.test_gpu_window import FAR, compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ranks,late_every", [(5, 2), (1023, 7), (1024, 1), (1025, 3), (4100, 1), (16383, 5), (16384, 9), (16390, 9)])
def test_many_flagged_ranks(ranks, late_every):
    from paper_2605_04478_amd import ccld
    # rings of four consecutive ranks; in every round one member of a flagged ring enters late
    rings = [[r, r + 1, r + 2, r + 3] for r in range(0, ranks - 3)][::3] or [list(range(ranks))]
    topo = tg.make_topology(ranks, rings)
    rng = np.random.default_rng(ranks)
    rows = []
    for c, mem in enumerate(rings):
        for s in range(3):
            late = mem[(c + s) % 4] if (c + s) % late_every == 0 else -1
            for r in mem:
                te = T0 + s * 10**7 + int(rng.integers(0, 50)) + (400_000 + int(rng.integers(0, 3)) if r == late else 0)
                rows.append((r, c, s, 0, 1 << 20, te, te + 100_000))
    cols = toy_cols(rows)
    p = rng.permutation(len(rows))
    cols = {k: v[p] for k, v in cols.items()}
    an = ccld.Analyzer(topo, max_window_records=len(rows))
    an.ingest(an.to_device(cols))
    g, ref = an.analyze_window(FAR, n_records=len(rows), per_record=True), orc.Oracle(topo).analyze_window(cols, FAR)
    assert g.n_flag > 0
    compare(g, ref, *an.rank_blame(), what=f"{ranks} ranks")
    an.close()
