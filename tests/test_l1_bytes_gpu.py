"""L1 searches whose pairs pass a filter of byte sums first, against the CPU oracle: the edges of its
tiles (64 points, 64 queries per wave and lane slot, 16 coordinates per chunk, 16 buffered points),
values far outside the sampled scale, ties, infinities and NaN.

A pair is dropped only on a lower bound of its distance, and the kept ones get the fp32 key that the
kernel without the filter gives them, so the first columns of a search with k > 64, which goes there,
must be the same bits.
"""
import numpy as np
import pytest

import workloads as W
from parity import check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def K():
    import paper_2206_14148_amd as K
    assert torch.cuda.is_available(), "these tests need the GPU"
    K.load()
    return K


def search(K, Q, X, k, plain=False, filtered=None):
    """filtered: whether the lists have to be the filter's.  (The kernel without it works on transposed
    queries, which then lie where the filter keeps its scale.)"""
    kk = 65 if plain else k
    plan = K.knn_plan(Q.shape[0], X.shape[0], Q.shape[1], kk, 256 * W.MB, "l1")
    assert plan.q_chunks == 1
    ws = torch.full((plan.workspace_bytes,), 0xA5, dtype=torch.uint8, device="cuda")
    idx, dist = K.knn_search(Q, X, kk, 256 * W.MB, metric="l1", workspace=ws)
    torch.cuda.synchronize()
    transposed = torch.equal(ws[:16].view(torch.float32).view(torch.int32), Q[0, :4].clone().view(torch.int32))
    print("filtered", not transposed, flush=True)
    if filtered is not None:
        assert transposed != filtered
    return idx[:, :k].cpu().numpy(), dist[:, :k].cpu().numpy()


def data(seed, m, n, d, kind):
    g = np.random.Generator(np.random.PCG64(seed))
    Q = g.standard_normal((m, d)).astype(np.float32)
    X = g.standard_normal((n, d)).astype(np.float32)
    if kind == "clusters":  # much narrower than a unit of the scale
        c = 100.0 * g.standard_normal((50, d)).astype(np.float32)
        X = c[g.integers(0, 50, n)] + np.float32(0.01) * X
        Q = c[g.integers(0, 50, m)] + np.float32(0.01) * Q
    elif kind == "many_clusters":  # the same, but a query's own cluster is less than the filter may let through
        c = 100.0 * g.standard_normal((500, d)).astype(np.float32)
        X = c[g.integers(0, 500, n)] + np.float32(0.01) * X
        Q = c[g.integers(0, 500, m)] + np.float32(0.01) * Q
    elif kind == "gmm":     # clusters as wide as they are apart
        c = 2.0 * g.standard_normal((100, d)).astype(np.float32)
        X += c[g.integers(0, 100, n)]
        Q += c[g.integers(0, 100, m)]
    elif kind == "outliers":  # a few points with values far outside the scale, and beyond 1e30
        X[g.integers(0, n, 50), g.integers(0, d, 50)] *= 100
        X[g.integers(0, n, 20), g.integers(0, d, 20)] = 1e32
    elif kind == "tails":   # some values far outside the sample's range, others beyond 1e30
        X *= np.exp(3.0 * g.standard_normal((n, d))).astype(np.float32)
        X[g.integers(0, n, 20), g.integers(0, d, 20)] = 1e32
    elif kind == "offset":
        Q += 1000.0
        X += 1000.0
    elif kind == "ties":
        Q, X = np.rint(Q), np.rint(X)
    elif kind == "equal":
        Q[:], X[:] = 2.5, 2.5
    return Q, X


# and whether the filter answers (where it would let too much through it says so, and the kernel without it
# makes the lists)
CASES = [(129, 4096, 16, 1, "normal", True), (257, 30_001, 17, 10, "normal", True), (1025, 30_003, 100, 10, "normal", True),
         (700, 31_001, 100, 10, "clusters", False), (700, 31_001, 100, 10, "many_clusters", True),
         (300, 30_000, 33, 7, "tails", False), (300, 30_000, 33, 7, "outliers", True),
         (513, 50_100, 185, 16, "normal", False), (513, 50_100, 185, 16, "gmm", True),
         (100, 196_000, 192, 64, "offset", False), (100, 196_000, 192, 64, "gmm", True), (300, 30_000, 16, 7, "offset", True),
         (2000, 51_191, 20, 17, "ties", True), (150, 30_159, 64, 10, "equal", False),
         (11_000, 9200, 128, 3, "normal", True), (140, 70_000, 57, 5, "normal", True), (300, 30_011, 16, 2, "normal", True),
         (1, 10_000, 24, 1, "normal", True), (64, 50_000, 5, 8, "normal", True), (65, 15_007, 9, 5, "tails", False),
         (65, 15_007, 9, 5, "outliers", True), (1500, 12_000, 8, 4, "normal", True)]


@pytest.mark.parametrize("m,n,d,k,kind,filtered", CASES)
def test_matches_oracle_and_the_search_without_the_filter(K, oracle, m, n, d, k, kind, filtered):
    print("case", m, n, d, k, kind, flush=True)
    Q, X = data(m + d, m, n, d, kind)
    Qd, Xd = torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda()
    idx, dist = search(K, Qd, Xd, k, filtered=filtered)
    idx0, dist0 = search(K, Qd, Xd, k, plain=True, filtered=False)
    assert np.array_equal(idx, idx0) and np.array_equal(dist, dist0)
    if kind not in ("tails", "outliers"):  # (1e32 sums leave the oracle's error bound for fp32 keys meaningless)
        rows = np.unique(np.linspace(0, m - 1, 60).astype(np.int64))
        o_idx, o_dist, o_next = oracle.knn(Q, X, k, rows=rows, metric="l1")
        check(idx[rows], dist[rows], o_idx, o_dist, o_next, n)


def test_infinities_nan_and_strided_rows(K):
    n = 15_000
    Q, X = data(5, 300, n, 36, "normal")
    X[7, 3] = np.inf
    X[8, 4] = -np.inf
    X[9, :] = np.nan
    Q[11, 0] = np.nan
    Q[12, 35] = np.inf
    Xw, Qw = torch.zeros(n, 39).cuda(), torch.zeros(300, 37).cuda()
    Xw[:, :36] = torch.from_numpy(X).cuda()
    Qw[:, :36] = torch.from_numpy(Q).cuda()
    idx, dist = search(K, Qw[:, :36], Xw[:, :36], 5, filtered=True)
    idx0, dist0 = search(K, Qw[:, :36], Xw[:, :36], 5, plain=True)
    assert np.array_equal(idx, idx0) and np.array_equal(dist, dist0, equal_nan=True)
    finite = np.ones(300, bool)
    finite[11:13] = False
    assert not np.isin(idx, (7, 8, 9))[finite].any()
