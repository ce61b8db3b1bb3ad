"""Haralick's f3 (correlation), f12 and f13 where the moments about 0 cancel:
marginals that lie apart, nearly all counts in one corner bin, up to 4e9 of
them, on every kernel (N <= 16, <= 32, above, above with many matrices)."""

import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1710_06189_amd as G  # noqa: E402

pytestmark = pytest.mark.gpu

# two roundings to fp32 (the result and, at worst, one ulp on top of it)
RTOL = 2.0 ** -23


def f3(P):
    """The correlation from whole-number moments."""
    N = len(P)
    c = [[int(v) for v in r] for r in P]
    T = sum(map(sum, c))
    rows, cols = [sum(r) for r in c], [sum(c[i][j] for i in range(N)) for j in range(N)]
    si, sj = sum(i * v for i, v in enumerate(rows)), sum(j * v for j, v in enumerate(cols))
    vi = T * sum(i * i * v for i, v in enumerate(rows)) - si * si
    vj = T * sum(j * j * v for j, v in enumerate(cols)) - sj * sj
    cov = T * sum(i * j * c[i][j] for i in range(N) for j in range(N) if c[i][j]) - si * sj
    return 1.0 if vi == 0 or vj == 0 else cov / (math.sqrt(vi) * math.sqrt(vj))


def corner(N, T, kind):
    """T counts in one bin of the top right corner and a few beside it."""
    P = np.zeros((N, N), dtype=np.uint32)
    if kind == "weak":
        P[0, N - 2], P[1, N - 2], P[0, N - 1], P[1, N - 1] = T, 2, 3, 1
    elif kind == "equal":  # fully correlated
        P[0, N - 2], P[1, N - 1] = T, 5
    elif kind == "opposite":
        P[0, N - 1], P[1, N - 2], P[1, N - 1] = T, 2, 2
    elif kind == "far":  # one count far from the others: a small covariance beside a large variance
        P[:, N // 2] = T // N
        P[N - 1, N // 2 + 1] = 1
    else:  # lower left: the other sign of i - j
        P[N - 1, 0], P[N - 2, 0], P[N - 1, 1], P[N - 2, 1] = T, 7, 1, 9
    return P


def run(mats):
    t = torch.from_numpy(np.stack(mats).view(np.int32)).cuda().view(torch.uint32)
    return G.glcm_haralick(t).cpu().numpy()


@pytest.mark.parametrize("N", [4, 15, 16, 17, 32, 33, 96, 256, 1024])
@pytest.mark.parametrize("T", [10 ** 6, 4 * 10 ** 9])
def test_correlation_of_marginals_that_lie_apart(N, T):
    kinds = ["weak", "equal", "opposite", "far", "lower"]
    mats = [corner(N, T, k) for k in kinds]
    want = np.array([f3(P) for P in mats])
    np.testing.assert_allclose(run(mats)[:, 2], want, rtol=RTOL)
    if N <= 96:  # many matrices: fewer wavefronts each
        got = run(mats * 60)[:, 2].reshape(60, len(kinds))
        np.testing.assert_allclose(got, np.broadcast_to(want, got.shape), rtol=RTOL)


@pytest.mark.parametrize("N", [5, 16, 31, 32, 40, 200])
def test_a_single_row_or_column_is_independent(N):
    """One occupied level in a marginal: p = px py, so f3 = 1, f12 = f13 = 0."""
    rng = np.random.default_rng(N)
    a, b = np.zeros((2, N, N), dtype=np.uint32)
    a[N // 3] = rng.integers(0, 1000, N)
    b[:, N - 1] = rng.integers(0, 1000, N)
    got = run([a, b])
    assert (got[:, 2] == 1.0).all() and (got[:, 11] == 0.0).all() and (got[:, 12] == 0.0).all()
