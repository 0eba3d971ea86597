"""Low-dimensional search through the octree: bit for bit what the vector-ALU path gives, which
looks at every pair."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def K():
    import paper_2206_14148_amd as K
    assert torch.cuda.is_available(), "these tests need the GPU"
    K.load()
    return K


def both(K, Q, X, k, limit=256 * W.MB):
    m, d = Q.shape
    n = X.shape[0]
    plan = K.knn_plan(m, n, d, k, limit)
    assert plan.path == K.KNN_PATH_LOWD_BF16 and plan.seed_cells >= 2
    bare = plan.min_limit_bytes + 8 * k * 256
    assert K.knn_plan(m, n, d, k, bare).path == K.KNN_PATH_LOWD
    idx, dist = K.knn_search(Q, X, k, limit)
    ref_idx, ref_dist = K.knn_search(Q, X, k, bare)
    torch.cuda.synchronize()
    assert torch.equal(idx, ref_idx) and torch.equal(dist, ref_dist)
    return idx


def points(kind, rows, d, gen):
    if kind == "normal":
        return torch.randn(rows, d, generator=gen, device="cuda")
    if kind == "far":  # a long way from the origin: neighbouring values are few roundings apart
        return 1000.0 + torch.rand(rows, d, generator=gen, device="cuda")
    if kind == "lattice":  # ties everywhere, points on the cells' borders, many of them equal
        return torch.randint(0, 9, (rows, d), generator=gen, device="cuda").float() / 8
    if kind == "clumps":  # dense clumps in an empty box
        c = torch.rand(20, d, generator=gen, device="cuda") * 100
        return c[torch.randint(0, 20, (rows,), generator=gen, device="cuda")] + \
            1e-2 * torch.randn(rows, d, generator=gen, device="cuda")
    if kind == "one_spot":  # all but one point in one cell: the filter path answers
        x = 1e-6 * torch.rand(rows, d, generator=gen, device="cuda")
        x[7] = 1e6
        return x
    return torch.rand(rows, d, generator=gen, device="cuda")


# list lengths around the register lists' (8, 16, 32) and the first beyond; fewest points and one less;
# fewest queries (one for eight points) and one less; queries that leave a wave, a workgroup or the
# eighth of the launch ragged
@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("kind,m,n,k", [
    ("uniform", 512, 4096, 1), ("uniform", 511, 4096, 1), ("uniform", 600, 4095, 8), ("uniform", 1025, 4097, 9),
    ("normal", 5000, 30_011, 16), ("normal", 9000, 50_000, 17), ("far", 5777, 20_000, 32), ("uniform", 5000, 20_000, 33),
    ("lattice", 12_049, 40_000, 12), ("clumps", 8000, 40_000, 16), ("one_spot", 7000, 20_000, 5),
    ("uniform", 70_000, 5_000, 3)])
def test_same_as_every_pair(K, d, kind, m, n, k):
    print("case", d, kind, m, n, k, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d * 1000 + m + k)
    X = points(kind, n, d, gen)
    # queries among the points, some outside their box
    Q = points(kind, m, d, gen) * 1.25 - 0.125
    both(K, Q, X, k)
    wide = torch.full((m, d + 2), 5.0, device="cuda")
    wide[:, :d] = Q
    both(K, wide[:, :d], X, k)


@pytest.mark.parametrize("d", [1, 2, 3])
def test_points_as_their_own_queries(K, d):
    # the order of the points serves the queries; a copy of them goes through an order of its own
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    X = points("normal", 20_001, d, gen)
    idx = both(K, X, X, 4)
    # the first neighbour is the point itself, or an equal one of lower index (on a line two of 20001
    # floats are equal now and then)
    assert torch.equal(X[idx[:, 0].long()], X)
    assert torch.equal(idx, both(K, X.clone(), X, 4))
    both(K, X[100:9000], X, 16)


def test_query_chunks_share_one_tree(K):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    X = points("uniform", 60_000, 2, gen)
    Q = points("uniform", 40_001, 2, gen)
    base = K.knn_plan(40_001, 60_000, 2, 16, 1 << 40)
    limit = base.norms_bytes + base.private_bytes + 2 * 2 * 10_000 * 16 * 4
    plan = K.knn_plan(40_001, 60_000, 2, 16, limit)
    assert plan.q_chunks > 2 and plan.seed_cells >= 2 and plan.chunk_rows >= 60_000 // 8
    both(K, Q, X, 16, limit)
    spot = points("one_spot", 60_000, 2, gen)  # several chunks on the filter path behind the tree's check
    both(K, Q, spot, 16, limit)


@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("k", [1, 5, 32])
def test_keys_beyond_the_largest_float_enter_no_list(K, d, k):
    # as on the path that looks at every pair: a pair whose fp32 distance is infinite is no neighbour
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * d + k)
    X, Q = points("uniform", 20_000, d, gen), points("uniform", 6000, d, gen)
    far = Q.clone()
    for i, v in enumerate((1e19, -1e19, 1.8446742e19, 3e19, 1e20, -1e25, 1e30, 3e38, -3e38)):
        far[7 * i + 3, i % d] = v
        far[2000 + i] = v
    idx = both(K, far, X, k)
    assert (idx[2004] == 2 ** 31 - 1).all()
    for scale in (1e-28, 1e-25, 1e-20, 1e-19, 1e18, 1e19, 1e20, 1e25, 1e37):
        print("scale", scale, flush=True)
        both(K, Q * scale, X * scale, k)


@pytest.mark.parametrize("m", [8000, 8007, 8191])
def test_queries_that_share_few_cells(K, m):
    # counted by one atomic for all lanes of a cell: whole waves, the ragged last one, a few cells and many
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)
    X = points("uniform", 30_000, 3, gen)
    Q = points("uniform", m, 3, gen)
    both(K, Q + 10, X, 16)
    mixed = Q.clone()
    mixed[::2] += 10
    mixed[1::8] -= 10
    both(K, mixed, X, 16)
