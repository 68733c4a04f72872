"""FDBSCAN with wide neighbourhoods: DM distances beyond the rows that there are,
joins that fall behind the levels and go over to a lane a row.  Labels, cluster
count and query count equal the oracle's sequential FDBSCAN."""
import numpy as np
import pytest
import torch

import oracle

from gpu_util import api

pytestmark = pytest.mark.gpu


def _list(n, rows, span):
    A = api()
    rng = np.random.default_rng(n)
    key = np.unique(rng.integers(0, rows * span, n))
    rec = np.zeros(len(key), A.CANDIDATE_DTYPE)
    rec["dm_index"], rec["sample"] = key // span, key % span
    rec["snr"] = (6.0 + 2.0 * rng.random(len(key))).astype(np.float32)
    return rec, torch.from_numpy(rec.view(np.uint8).copy()).cuda()


@pytest.mark.parametrize("n,rows,span,te,de,mp", [
    (3000, 200, 400, 3, 199, 5),       # every row in reach: 399 rows a neighbourhood
    (3000, 200, 400, 3, 100, 60),      # some points core, most not
    (2000, 30, 900, 4, 11, 4),         # 23 rows a neighbourhood: taken in turn
    (2000, 30, 900, 4, 12, 4),         # 25: from the counter
    (1500, 64, 6000, 2, 63, 2),        # many small clusters
    (1200, 32, 90, 40, 31, 4),         # one cloud, long runs
    (700, 1, 3000, 5, 65535, 3),       # one row
    (40, 5, 50, 3, 70, 3),
    (900, 30, 400, 3, 30, 4),
])
def test_equals_sequential(n, rows, span, te, de, mp):
    rec, buf = _list(n, rows, span)
    labels, nc, nq = api().fdbscan_candidates(buf, len(rec), rows, te, de, 2.0, mp)
    want, kc, kq = oracle.fdbscan(rec["sample"], rec["dm_index"], rec["snr"], te, de, 2.0, mp)
    assert (int(nc.item()), int(nq.item())) == (kc, kq)
    assert np.array_equal(labels.cpu().numpy(), want)


def _ms(f):
    f()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = 1e9
    for _ in range(3):
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_rows_out_of_reach_cost_nothing():
    """A DM distance beyond the rows that there are reaches what the last row's
    does, and takes as long (it took 70 times that)."""
    A = api()
    rec, buf = _list(2400, 64, 8000)
    last, beyond = (_ms(lambda: A.fdbscan_candidates(buf, len(rec), 64, 16, de, 2.0, 5)) for de in (63, 10000))
    assert beyond < 1.5 * last


def test_wide_joins_keep_the_lanes_busy():
    """Expanding 4090 points with all 400 rows in reach against DBSCAN of the
    same list on the whole GPU: 10 times as long, 12 before joins went by groups
    of lanes, 49 with groups alone."""
    A = api()
    rec, buf = _list(6000, 400, 4000)
    args = (buf, len(rec), 400, 4, 399, 2.0, 5)
    assert _ms(lambda: A.fdbscan_candidates(*args)) < 24 * _ms(lambda: A.cluster_candidates(*args))
