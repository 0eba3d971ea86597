"""Rows that are not whole groups of four coordinates, and rows that begin at any multiple of 4 bytes, on every path
for d > 8 and the cosine metric: same neighbours and distances as the oracle, and no read outside the rows (guard
values around them are NaN, which would show)."""
import numpy as np
import pytest

import workloads as W
from parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def spread(a, before, after):
    """The rows of a on the device, `before` and `after` NaNs around each."""
    wide = torch.full((len(a), before + a.shape[1] + after), float("nan"), device="cuda")
    wide[:, before:before + a.shape[1]] = torch.from_numpy(a).cuda()
    return wide[:, before:before + a.shape[1]]


# (m, n, d, k, metric): path 6 (d from 17 to 256), path 7 (lists staged in the stops), path
# 5 (k = 1 of 300 queries; with a range per compute unit and with fewer), few queries; the cosine metric with fewer coordinates than one group, and on path 6
CASES = [(70, 66_000, 21, 9, "l2"), (130, 66_000, 50, 100, "l2"), (70, 66_000, 131, 10, "l2"), (130, 66_000, 255, 3, "l2"),
         (40, 66_000, 301, 12, "l2"), (300, 66_000, 259, 1, "l2"), (20, 66_000, 514, 2, "l2"), (130, 66_000, 514, 2, "l2"), (70, 66_000, 200, 5, "l2"),
         (700, 5_000, 30, 40, "l2"), (300, 3_000, 515, 300, "l2"), (5, 3_000, 33, 10, "l2"), (3, 1_000, 35, 4, "l2"),
         (50, 900, 1, 7, "cosine"), (50, 900, 3, 7, "cosine"), (80, 66_000, 3, 9, "cosine"), (80, 66_000, 46, 9, "cosine"), (80, 66_000, 46, 5, "cosine")]


@pytest.mark.parametrize("before,after", [(0, 0), (1, 0), (0, 3)])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "m%d_n%d_d%d_k%d_%s" % c)
def test_matches_oracle(oracle, case, before, after):
    import paper_2206_14148_amd as K

    m, n, d, k, metric = case
    print("case", case, before, after, flush=True)
    rng = np.random.default_rng(d * 7 + n)
    X = rng.standard_normal((n, d), dtype=np.float32)
    Q = rng.standard_normal((m, d), dtype=np.float32)
    Xd, Qd = spread(X, before, after), spread(Q, after, before)
    idx, dist = K.knn_search(Qd, Xd, k, W.GB, metric=metric)
    torch.cuda.synchronize()
    rows = np.arange(0, m, max(1, m // 40))
    o_idx, o_dist, o_next = oracle.knn(Q, X, k, rows=rows, metric=metric)
    check(idx.cpu().numpy()[rows], dist.cpu().numpy()[rows], o_idx, o_dist, o_next, n)
    assert torch.isfinite(dist).all()
