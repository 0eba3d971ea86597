"""Small searches evaluate every pair: bit for bit the results of the filter paths, which the same
call takes as a part of a larger one."""
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


# rows that are 16-byte aligned and not; a row's length at the ends of the staged pieces of 32 and of the
# groups of 8 and 4; one point, one wave's worth and one more; queries that leave a group of four;
# lists of one, of a wave and of the longest kept here
@pytest.mark.parametrize("m,n,d,k", [
    (1, 1, 9, 1), (3, 64, 9, 10), (4, 65, 12, 64), (5, 1000, 31, 65), (17, 5000, 32, 10), (9, 20_011, 33, 7),
    (16, 20_000, 50, 10), (63, 3001, 63, 5), (64, 3001, 64, 128), (65, 2999, 65, 33), (2, 70_001, 100, 100),
    (1, 70_000, 257, 10), (7, 1500, 300, 16), (300, 4000, 16, 10)])
def test_same_as_the_filter_paths(K, oracle, m, n, d, k):
    from parity import check
    print("case", m, n, d, k, flush=True)
    Q, X = W.random_case(8800 + m + d, m, n, d)
    Qd, Xd = torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda()
    idx, dist = K.knn_search(Qd, Xd, k, W.GB)
    Xw = torch.full((n, d + 3), 7.0, device="cuda")
    Xw[:, :d] = Xd
    s_idx, s_dist = K.knn_search(Qd, Xw[:, :d], k, W.GB)
    # the smallest limit: short lists, as many ranges as fit
    t_idx, t_dist = K.knn_search(Qd, Xd, k, K.knn_plan(m, n, d, k, W.GB).min_limit_bytes)
    # the same queries among so many that the filters answer
    more = int(5.1e9 / (n * (d + 16))) + 1
    if more < 200_000:
        big = torch.cat([Qd, Xd[:1].expand(more, d)]).contiguous()
        b_idx, b_dist = K.knn_search(big, Xd, k, 8 * W.GB)
    torch.cuda.synchronize()
    o_idx, o_dist, o_next = oracle.knn(Q, X, k)
    check(idx.cpu().numpy(), dist.cpu().numpy(), o_idx, o_dist, o_next, n)
    assert torch.equal(idx, s_idx) and torch.equal(dist, s_dist)
    assert torch.equal(idx, t_idx) and torch.equal(dist, t_dist)
    if more < 200_000:
        assert torch.equal(idx, b_idx[:m]) and torch.equal(dist, b_dist[:m])


def test_equal_points_keep_the_lowest_indices(K):
    X = torch.full((30_000, 20), 0.75, device="cuda")
    idx, dist = K.knn_search(X[:6] + 0.5, X, 9, W.GB)
    torch.cuda.synchronize()
    assert (idx == torch.arange(9, device="cuda", dtype=torch.int32)).all() and (dist == 5.0).all()


# hundreds of lists a query, merged from the lanes' first entries up to k = 52: neighbours spread over the lists, all in
# one of them, at one place of every list (multiples of the stride of a lane's entries), and equal ones
@pytest.mark.parametrize("k", [1, 2, 10, 51, 52, 53, 64])
@pytest.mark.parametrize("place", ["spread", "one", "stride", "equal"])
def test_merge_of_many_lists(K, oracle, k, place):
    from parity import check
    m, n, d = 3, 150_001, 12
    print("case", k, place, flush=True)
    Q, X = W.random_case(8900 + k, m, n, d)
    near = {"one": slice(777, 777 + 40), "stride": slice(5, n, 4096)}.get(place)
    if near is not None:
        X[near] *= 1e-3
        Q *= 1e-3
    if place == "equal":
        Q, X = Q.round(), X.round()
    Qd, Xd = torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda()
    idx, dist = K.knn_search(Qd, Xd, k, W.GB)
    t_idx, t_dist = K.knn_search(Qd, Xd, k, K.knn_plan(m, n, d, k, W.GB).min_limit_bytes)
    torch.cuda.synchronize()
    o_idx, o_dist, o_next = oracle.knn(Q, X, k)
    check(idx.cpu().numpy(), dist.cpu().numpy(), o_idx, o_dist, o_next, n)
    assert torch.equal(idx, t_idx) and torch.equal(dist, t_dist)


# a few entries a lane, and their line to the lanes' first ones (three runs of 512 entries, or k / 8); k that divide 512, whose
# entries of a lane would be of one place, and others
@pytest.mark.parametrize("m,n,k", [(1, 16_000, 8), (3, 50_001, 8), (2, 23_041, 16), (1, 13_000, 32), (18, 60_000, 32),
                                   (5, 10_000, 44), (3, 40_000, 44), (4, 100_003, 48), (1, 33_000, 2)])
def test_merge_where_a_lane_has_few_entries(K, oracle, m, n, k):
    from parity import check
    print("case", m, n, k, flush=True)
    Q, X = W.random_case(9000 + k, m, n, 16)
    idx, dist = K.knn_search(torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda(), k, W.GB)
    torch.cuda.synchronize()
    o_idx, o_dist, o_next = oracle.knn(Q, X, k)
    check(idx.cpu().numpy(), dist.cpu().numpy(), o_idx, o_dist, o_next, n)
