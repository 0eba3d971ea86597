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


GRID_WORD, LEFT_WORD = 32, 33  # header words: the tree serves the call; waves of the last chunk that gave up


def both(K, Q, X, k, limit=256 * W.MB, tree=None, left=None):
    """The call against the path that looks at every pair; whether the tree answers it (tree) and
    leaves some waves to the filter (left) where that is expected."""
    m, d = Q.shape
    n = X.shape[0]
    plan = K.knn_plan(m, n, d, k, limit)
    assert plan.path == K.KNN_PATH_LOWD_BF16 and plan.seed_cells >= 2
    bare = plan.min_limit_bytes + 8 * k * 256
    assert K.knn_plan(m, n, d, k, bare).path == K.KNN_PATH_LOWD
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
    idx, dist = K.knn_search(Q, X, k, limit, workspace=ws)
    ref_idx, ref_dist = K.knn_search(Q, X, k, bare)
    torch.cuda.synchronize()
    header = ws[:256].view(torch.int32)
    print("tree", int(header[GRID_WORD]), "left", int(header[LEFT_WORD]), "of", (m + 63) // 64, flush=True)
    assert torch.equal(idx, ref_idx) and torch.equal(dist, ref_dist)
    if tree is not None:
        assert int(header[GRID_WORD]) == tree
    if left is not None:
        assert (int(header[LEFT_WORD]) > 0) == left
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
    if kind == "fine_lattice":  # ties, points on the cells' borders, two or so to a cell
        return torch.randint(0, {1: 4096, 2: 64, 3: 16}[d], (rows, d), generator=gen, device="cuda").float() / 8
    if kind == "many_clumps":
        c = torch.rand(500, d, generator=gen, device="cuda") * 100
        return c[torch.randint(0, 500, (rows,), generator=gen, device="cuda")] + \
            1e-3 * torch.randn(rows, d, generator=gen, device="cuda")
    if kind == "shell":
        x = torch.randn(rows, d, generator=gen, device="cuda")
        return x / x.norm(dim=1, keepdim=True)
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


# the same where the tree is known to answer (or to turn the points down): twice as many queries as points
@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("kind,m,n,k,tree", [
    ("uniform", 8192, 4096, 1, 1), ("uniform", 8191, 4096, 8, 1), ("uniform", 8193, 4095, 8, 0), ("uniform", 8195, 4097, 9, 1),
    ("normal", 40_001, 20_000, 16, 1), ("normal", 40_063, 20_001, 17, 1), ("far", 16_000, 8000, 32, 1),
    ("uniform", 20_000, 8000, 33, 0), ("fine_lattice", 16_449, 8192, 12, 1), ("many_clumps", 16_321, 8000, 16, 1),
    ("one_spot", 16_000, 8000, 5, 0), ("uniform", 70_000, 5_000, 3, 1)])
def test_the_tree_answers(K, d, kind, m, n, k, tree):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d * 1000 + m + k)
    X = points(kind, n, d, gen)
    Q = points(kind, m, d, gen) * 1.0625 - 0.03125
    both(K, Q, X, k, tree=tree, left=False)
    wide = torch.full((m, d + 2), 5.0, device="cuda")
    wide[:, :d] = Q
    both(K, wide[:, :d], X, k, tree=tree, left=False)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("k", [1, 16, 32])
def test_queries_the_tree_is_no_help_for(K, d, k):
    # waves that would look through much of the tree leave their rows, and no others, to the filter
    gen = torch.Generator(device="cuda")
    gen.manual_seed(10 * d + k)
    n, m = 20_000, 40_021
    S = points("shell", n, d, gen)
    centre = 1e-3 * points("normal", m, d, gen)
    both(K, centre, S, k, tree=1, left=True)
    mixed = points("shell", m, d, gen)
    mixed[::3] *= 1e-3
    both(K, mixed, S, k, tree=1, left=True)
    X, Q = points("uniform", n, d, gen), points("uniform", m, d, gen)
    both(K, Q, X, k, tree=1, left=False)
    Q[17_000], Q[m - 1, 0] = 1e6, -1e5
    both(K, Q, X, k, tree=1, left=True)
    both(K, Q + 1e5, X, k, tree=1, left=True)
    # beyond what the filter's sums hold the tree keeps the rows, beside others that it leaves
    Q[16_990:17_010:2] = 1e19
    both(K, Q, X, k, tree=1)


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
    both(K, X, X[:9000], 4, tree=1)  # the points are the first of the queries



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


def test_query_chunks_and_rows_left_by_one_of_them(K):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(10)
    X, Q = points("uniform", 5000, 2, gen), points("uniform", 80_001, 2, gen)
    base = K.knn_plan(80_001, 5000, 2, 16, 1 << 40)
    limit = base.norms_bytes + base.private_bytes + 2 * 2 * 11_000 * base.n_splits * 16 * 4
    plan = K.knn_plan(80_001, 5000, 2, 16, limit)
    print(plan.q_chunks, plan.chunk_rows, plan.n_splits, flush=True)
    assert plan.q_chunks > 3 and plan.seed_cells >= 2 and plan.chunk_rows >= 10_000
    both(K, Q, X, 16, limit, tree=1, left=False)
    Q[plan.chunk_rows + 100] = 1e6   # the second chunk leaves a wave; the filter has the area from then on
    both(K, Q, X, 16, limit, tree=0, left=False)
    Q[5] = 1e6                       # already the first
    both(K, Q, X, 16, limit, tree=0, left=False)
    Q[:] = points("uniform", 80_001, 2, gen)
    Q[80_000] = 1e6                  # only the last
    both(K, Q, X, 16, limit, tree=1, left=True)
    both(K, Q, points("one_spot", 5000, 2, gen), 16, limit, tree=0, left=False)


@pytest.mark.parametrize("d", [1, 2, 3])
@pytest.mark.parametrize("k", [1, 5, 32])
def test_keys_beyond_the_largest_float_enter_no_list(K, d, k):
    # as on the path that looks at every pair: a pair whose fp32 distance is infinite is no neighbour
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * d + k)
    X, Q = points("uniform", 8000, d, gen), points("uniform", 16_001, d, gen)
    far = Q.clone()
    for i, v in enumerate((1e19, -1e19, 1.8446742e19, 3e19, 1e20, -1e25, 1e30, 3e38, -3e38)):
        far[7 * i + 3, i % d] = v
        far[2000 + i] = v
    idx = both(K, far, X, k, tree=1)
    assert (idx[2004] == 2 ** 31 - 1).all()
    for scale in (1e-28, 1e-25, 1e-20, 1e-19, 1e18, 1e19, 1e20, 1e25, 1e37):
        print("scale", scale, flush=True)
        both(K, Q * scale, X * scale, k, tree=1)


@pytest.mark.parametrize("m", [8192, 8199, 8255])
def test_queries_that_share_few_cells(K, m):
    # counted by one atomic for all lanes of a cell: whole waves, the ragged last one, a few cells and many
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)
    X = points("uniform", 4096, 3, gen)
    Q = points("uniform", m, 3, gen)
    both(K, Q + 10, X, 16, tree=1)
    mixed = Q.clone()
    mixed[::2] += 10
    mixed[1::8] -= 10
    both(K, mixed, X, 16, tree=1)
