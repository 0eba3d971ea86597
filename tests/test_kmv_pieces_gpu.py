"""GPU tests of y = K v over fp16 pieces (9 to 64 coordinates): edges of chunks, tiles and ranges, rows and points out
of the pieces' range, against the fp64 oracle.

Tolerance (eps = 2^-24, c = 1 / (2 l^2)): a coordinate in exponent units is moved by at most 2 eps of itself or 2 eps,
so an exponent by 2 eps (|a| + |b|) (|a - b| + sqrt(d)), and by 4 eps where a product is left out; the sums of products and the norms round a few times at
(|a| + |b|)^2 / 2: together within (d + 8) eps (sqrt(c) (|x| + |z|) + 1)^2.  Sums of at most 64 entries in fp32 and
exp2's last bit add 4e-6 of the magnitudes."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


def run(X, Z, v, lengthscale, limit=W.GB, workspace=None):
    import paper_2206_14148_amd as K

    y = K.kmv_apply(*(torch.from_numpy(a).cuda() for a in (X, Z, v)), 1.5, lengthscale, limit, workspace=workspace)
    return y.cpu().numpy()


def bound(X, Z, v, lengthscale):
    X, Z, d = X.astype(np.float64), Z.astype(np.float64), X.shape[1]
    c = 0.5 / lengthscale ** 2
    tol = np.empty(len(X))
    for i, x in enumerate(X):
        mag = 1.5 * np.exp(-c * ((x - Z) ** 2).sum(1)) * np.abs(v)
        e = (np.sqrt(c) * (np.sqrt((x * x).sum()) + np.sqrt((Z * Z).sum(1))) + 1) ** 2
        tol[i] = (mag * (4e-6 + (d + 8) * EPS * e)).sum()
    return tol + 1e-37 * np.abs(v).sum()


# chunks of 16 coordinates; tiles of 128 points (64 above 32 coordinates); 128 rows of a workgroup; several ranges
CASES = [(1, 1, 9), (127, 127, 16), (128, 128, 17), (129, 129, 32), (130, 63, 33), (31, 64, 48), (33, 65, 49),
         (200, 193, 64), (40, 9_000, 20), (1_000, 2_500, 10)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n%d_m%d_d%d" % c)
@pytest.mark.parametrize("wide", [0.4, 1.5])
def test_matches_oracle(oracle, case, wide):
    import paper_2206_14148_amd as K

    n, m, d = case
    print("case", case, wide, flush=True)
    lengthscale = wide * d ** 0.5
    X, Z, v = W.random_kmv_case(n + d, n, m, d)
    want = K.load().kmv_workspace_bytes(n, m, d, lengthscale, W.GB)
    assert want > K.kmv_plan(n, m, d, W.GB).workspace_bytes
    buf = torch.full((want + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    y = run(X, Z, v, lengthscale, workspace=buf[:want])
    assert (buf[want:] == 0xA5).all()
    err, tol = np.abs(y - oracle.kmv(X, Z, v, 1.5, lengthscale)), bound(X, Z, v, lengthscale)
    print("  worst", float((err / tol).max()), flush=True)
    assert (err <= tol).all()
    assert np.array_equal(y, run(X, Z, v, lengthscale))


@pytest.mark.parametrize("far", [False, True], ids=["usual", "beside_a_far_point"])
def test_products_and_norms_are_of_the_same_points(far):
    # Everything up to the exponential is exact here: the lengthscale makes the unit of the pieces that of the
    # coordinates, 32 + 2^-6 takes both pieces, its square and the norms fit fp32.  The product of the low pieces is 2^-12:
    # left out of the products or of the norms alone it moves an entry by 1e-4.  exp2's last bit and the sum: 4 eps.
    d = 30
    X = np.zeros((d, d), np.float32)
    X[np.arange(d), np.arange(d)] = 32 + 2.0 ** -6
    Z = X.copy()
    Z[np.arange(d), (np.arange(d) + 1) % d] = 1.0
    v = np.ones(d, np.float32)
    lengthscale = float(np.sqrt(np.log2(np.e)))
    if far:  # the products of its tile are scaled back
        Z = np.concatenate([Z, np.full((1, d), 1e5, np.float32)])
        v = np.append(v, np.float32(1))
    assert np.allclose(run(X, X, np.ones(d, np.float32), lengthscale), 1.5, rtol=4 * EPS, atol=0)
    assert np.allclose(run(X, Z, v, lengthscale), 1.5 * 2.0 ** -0.5, rtol=4 * EPS, atol=0)


@pytest.mark.parametrize("d", [9, 16, 24, 32, 64])
@pytest.mark.parametrize("wide", [0.6, 1.5])
@pytest.mark.parametrize("mean", [0.0, 1.0, 10.0, 100.0])
def test_errors_are_those_of_six_products(oracle, d, wide, mean):
    """Against 64 bits, weights of one sign (a loss that all entries share does not average out): no more than the kernel
    that the plan's workspace leads to, whose six products of bf16 pieces are those of fp32.  Both errors are roundings
    that a seed draws: 1.15 for what is left of that over three seeds of 300 rows."""
    import paper_2206_14148_amd as K

    lengthscale, n, m = wide * d ** 0.5, 300, 2_000
    small = torch.empty(K.kmv_plan(n, m, d, W.GB).workspace_bytes, dtype=torch.uint8, device="cuda")
    assert small.numel() < K.load().kmv_workspace_bytes(n, m, d, lengthscale, W.GB)
    errors = np.zeros(2)
    for seed in range(3):
        rng = np.random.default_rng(seed)
        Z = (mean + rng.standard_normal((m, d))).astype(np.float32)
        v = (rng.random(m) + 0.5).astype(np.float32)
        ref = oracle.kmv(Z[:n], Z, v, 1.5, lengthscale)
        for i, ws in enumerate((small, None)):
            errors[i] += np.linalg.norm(run(Z[:n].copy(), Z, v, lengthscale, workspace=ws) - ref) / np.linalg.norm(ref)
    print("  six products %.2e  pieces %.2e" % tuple(errors / 3), flush=True)
    assert errors[1] <= 1.15 * errors[0]


@pytest.mark.parametrize("d", [12, 40])
def test_rows_and_points_out_of_range(oracle, d):
    # coordinates beyond 32768 exponent units: the products of their tile and of their rows are scaled back
    X, Z, v = W.random_kmv_case(77, 300, 500, d)
    X[40, 3], Z[200, d - 1], Z[201] = 1e6, -3e5, 4e4
    y = run(X, Z, v, 3.0)
    ref = oracle.kmv(X, Z, v, 1.5, 3.0)
    keep = np.arange(300) != 40
    near = np.ones(500, bool)
    near[[200, 201]] = False  # entries of exactly 0 for every row, out of the bound's formula
    assert y[40] == 0.0 and ref[40] == 0.0
    assert (np.abs(y - ref)[keep] <= bound(X[keep], Z[near], v[near], 3.0)).all()


@pytest.mark.parametrize("d", [9, 20, 40, 64])
def test_far_points_meet_themselves(d):
    # powers of two up to 2^59 units of the pieces, which all fit: an entry of a point with itself is exactly 1, however far,
    # beside rows and points that are in range, and every other one 0
    n = 300
    X = np.zeros((n, d), np.float32)
    X[np.arange(n), np.arange(n) * 7 % d] = 2.0 ** (6 + np.arange(n) * 11 % 54) * np.where(np.arange(n) // d % 2, 1, -1)
    X = np.unique(X, axis=0)
    v = np.random.default_rng(d).standard_normal(len(X)).astype(np.float32)
    y = run(X, X, v, float(np.sqrt(np.log2(np.e))))
    assert np.allclose(y, 1.5 * v.astype(np.float64), rtol=4 * EPS, atol=0)


@pytest.mark.parametrize("roomy", [True, False], ids=["pieces", "plan"])
@pytest.mark.parametrize("d", [9, 20, 64, 100])
def test_nans_show_and_infinite_coordinates_are_far(oracle, d, roomy):
    # as with up to 8 coordinates: a NaN row gives NaN, a NaN point makes every sum NaN, an entry of a point at
    # infinity with one that is not is 0; whatever the workspace
    import paper_2206_14148_amd as K

    X, Z, v = W.random_kmv_case(78, 300, 500, d)
    lengthscale = 0.5 * d ** 0.5
    size = (K.load().kmv_workspace_bytes(300, 500, d, lengthscale, W.GB) if roomy
            else K.kmv_plan(300, 500, d, W.GB).workspace_bytes)
    assert roomy or d > 64 or size < K.load().kmv_workspace_bytes(300, 500, d, lengthscale, W.GB)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    X[40, 3], X[41, 0], X[299, d - 1], Z[200, d - 1], Z[201] = np.nan, np.inf, -np.inf, -np.inf, np.inf
    y = run(X, Z, v, lengthscale, workspace=ws)
    keep, near = np.ones(300, bool), np.ones(500, bool)
    keep[[40, 41, 299]], near[[200, 201]] = False, False
    assert np.isnan(y[40]) and (y[[41, 299]] == 0).all()
    ref = oracle.kmv(X[keep], Z[near], v[near], 1.5, lengthscale)
    assert (np.abs(y[keep] - ref) <= bound(X[keep], Z[near], v[near], lengthscale)).all()
    Z[499, 1] = np.nan
    assert np.isnan(run(X, Z, v, lengthscale, workspace=ws)).all()
