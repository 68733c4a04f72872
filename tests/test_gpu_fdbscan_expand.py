"""FDBSCAN's expansion where its parts meet their edges: levels of more points
than the expanding wave takes at once, runs longer than a group reads at once,
rows shorter and longer than a group's probes, many starts within one scan
step and starts several steps apart, one DM row and hundreds.  Labels, cluster
count and query count equal the oracle's sequential FDBSCAN."""
import numpy as np
import pytest
import torch

import oracle

from gpu_util import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(n=3, rows=1, span=4, te=2, de=0, se=9.0, mp=2),
    dict(n=700, rows=1, span=300, te=40, de=0, se=0.5, mp=4),      # one row, runs of two hundred
    dict(n=900, rows=40, span=60, te=3, de=2, se=1.0, mp=4),       # one dense cloud: wide levels
    dict(n=1500, rows=300, span=80, te=2, de=30, se=0.3, mp=6),    # 61 DM rows a neighbourhood
    dict(n=3000, rows=30, span=6000, te=6, de=1, se=2.0, mp=3),    # hundreds of small clusters
    dict(n=9500, rows=64, span=60000, te=8, de=2, se=2.0, mp=4),   # few starts, scan steps apart
], ids=lambda k: f"n{k['n']}-rows{k['rows']}-de{k['de']}")
def test_equals_sequential(kw):
    A = api()
    rng = np.random.default_rng(kw["n"])
    key = np.unique(rng.integers(0, kw["rows"] * kw["span"], kw["n"]))
    rec = np.zeros(len(key), A.CANDIDATE_DTYPE)
    rec["dm_index"], rec["sample"] = key // kw["span"], key % kw["span"]
    rec["snr"] = (6.0 + 2.0 * rng.random(len(key))).astype(np.float32)
    buf = torch.from_numpy(rec.view(np.uint8).copy()).cuda()
    labels, nc, nq = A.fdbscan_candidates(buf, len(rec), kw["rows"], kw["te"], kw["de"], kw["se"], kw["mp"])
    want, kc, kq = oracle.fdbscan(rec["sample"], rec["dm_index"], rec["snr"], kw["te"], kw["de"], kw["se"], kw["mp"])
    assert (int(nc.item()), int(nq.item())) == (kc, kq)
    assert np.array_equal(labels.cpu().numpy(), want)
