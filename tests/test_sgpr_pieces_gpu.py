"""GPU tests of the SGPR sums over 16-bit pieces of K_uf: tile and stage edges, tiles split over workgroups, several
chunks, both kinds of pieces, against the definition in fp64 on the same GPU.

Tolerance (eps = 2^-24): an entry has relative error <= a (d + 4) eps + 2 eps, a its exponent (difference form,
hardware exp2); two fp16 pieces hold it to 2^-23 more and the products of the low pieces that are left out are below
2^-24, three bf16 pieces to 2^-26; sums run over 384 columns in fp32 (384 eps at most) and lose nothing beyond.  All
terms of A are positive, so |A - ref| <= A (2 (a (d + 4) + 2 + 3) + 384) eps; b is summed in fp64:
|b - ref| <= sum |K y| (a (d + 4) + 4) eps."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


def reference(U, X, y, variance, lengthscale):
    U, X, y = U.double(), X.double(), y.double()
    A = torch.zeros(len(U), len(U), dtype=torch.float64, device="cuda")
    b, mag = torch.zeros(2, len(U), dtype=torch.float64, device="cuda")
    worst = 0.0
    for s in range(0, len(X), 8192):
        sq = sum((U[:, t, None] - X[None, s:s + 8192, t]).square() for t in range(U.shape[1]))
        worst = max(worst, float(sq.max()))
        k = variance * torch.exp(sq * (-0.5 / lengthscale ** 2))
        A += k @ k.T.contiguous()
        b += k @ y[s:s + 8192]
        mag += k @ y[s:s + 8192].abs()
    return A, b, mag, 0.5 * worst / lengthscale ** 2


# (m, n, d, limit): one tile; tile edges; stage edges; a tile over many workgroups; several tiles of one set and of
# several; many coordinates; chunks (the limit holds some of the columns)
CASES = [(1, 1, 1, W.GB), (127, 15, 2, W.GB), (128, 16, 3, W.GB), (129, 17, 4, W.GB), (100, 257, 16, W.GB),
         (64, 20_001, 3, W.GB), (300, 4_095, 17, W.GB), (1_025, 3_000, 5, W.GB), (2_100, 1_111, 2, W.GB),
         (257, 60_001, 2, 80 * W.MB), (1_500, 9_000, 1, 80 * W.MB)]


@pytest.mark.parametrize("wide", [False, True], ids=["two_pieces", "three_pieces"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "m%d_n%d_d%d" % c[:3])
def test_sums_match_the_definition(case, wide):
    import paper_2206_14148_amd as K

    m, n, d, limit = case
    print("case", case, wide, flush=True)
    plan = K.sgpr_plan(m, n, d, limit)
    want = K.sgpr_workspace_bytes(m, n, d, limit)
    assert plan.workspace_bytes <= want <= limit
    gen = torch.Generator(device="cuda").manual_seed(m + n)
    U = torch.rand(m, d, generator=gen, device="cuda")
    X = torch.rand(n, d, generator=gen, device="cuda")
    y = torch.randn(n, generator=gen, device="cuda")
    # radius(U) + radius(X) is at most 2 sqrt(d): entries of 2^-12 and more, or far below
    lengthscale = d ** 0.5 * (0.5 if not wide else 0.1)
    buf = torch.full((want + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    A, b = K.sgpr_accumulate(U, X, y, 1.3, lengthscale, limit, workspace=buf[:want])
    assert (buf[want:] == 0xA5).all()
    ref, rb, mag, a = reference(U, X, y, 1.3, lengthscale)
    assert torch.equal(A, A.T)
    tol = ref * (2 * (a * (d + 4) + 5) + 384) * EPS + 1e-37 * n
    print("  worst A", float(((A - ref).abs() / tol).max()), "b", float(((b - rb).abs() / (mag * EPS)).max()), flush=True)
    assert ((A - ref).abs() <= tol).all()
    assert ((b - rb).abs() <= mag * (a * (d + 4) + 4) * EPS + 1e-37 * n).all()
    A2, b2 = K.sgpr_accumulate(U, X, y, 1.3, lengthscale, limit)  # a fixed order, whatever the workspace held
    assert torch.equal(A, A2) and torch.equal(b, b2)


def test_a_nan_stays_in_its_rows():
    import paper_2206_14148_amd as K

    U, X, y = (torch.from_numpy(v).cuda() for v in W.random_sgpr_case(3, 200, 3000, 3))
    U[7, 1] = float("nan")
    A, b = K.sgpr_accumulate(U, X, y, 1.0, 3.0, W.GB)
    rows = torch.arange(200, device="cuda") != 7
    U[7, 1] = 0.0
    ref, rb, _, _ = reference(U, X, y, 1.0, 3.0)
    assert A[7].isnan().all() and A[:, 7].isnan().all() and b[7].isnan()
    assert np.allclose(A[rows][:, rows].cpu(), ref[rows][:, rows].cpu(), rtol=1e-4, atol=0)
    assert np.allclose(b[rows].cpu(), rb[rows].cpu(), rtol=1e-4, atol=1e-3)
