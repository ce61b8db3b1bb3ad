"""The maximal correlation coefficient at the edges of its 16 x 16 tiles, on
spectra whose largest eigenvalue repeats, and at the largest counts."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402

pytestmark = pytest.mark.gpu


def near_diagonal(K, N, seed, top=200):
    g = np.random.Generator(np.random.PCG64(seed))
    d = np.abs(np.subtract.outer(np.arange(N), np.arange(N)))
    return (g.integers(0, top, size=(K, N, N)) * np.exp(-d / max(1.0, N / 6.0))).astype(np.uint32)


def blocks(N, parts):
    """`parts` independent blocks: the eigenvalue 1 occurs `parts` times."""
    P = np.zeros((1, N, N), dtype=np.uint32)
    for b in np.array_split(np.arange(N), parts):
        P[0][np.ix_(b, b)] = 3 + b[0]
    return P


CASES = [(f"N={N}", near_diagonal(5, N, N)) for N in (1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64)] + [
    ("two blocks", blocks(20, 2)), ("four blocks", blocks(40, 4)),
    ("largest counts", np.full((1, 64, 64), 2 ** 32 - 1, dtype=np.uint32) - near_diagonal(1, 64, 7)),
    ("more matrices than wavefronts", near_diagonal(20011, 3, 9)),
]


@pytest.mark.parametrize("name,P", CASES, ids=[c[0] for c in CASES])
def test_mcc_tiles(name, P):
    """2e-7 relative for the fp32 store, 1e-6 absolute for the oracle's own
    error near 0 (the square root of an eigenvalue off by about 1e-13)."""
    got = G.glcm_haralick_mcc(torch.from_numpy(P.view(np.int32)).cuda().view(torch.uint32)).cpu().numpy().astype(np.float64)
    want = oracle.haralick_mcc(P[:64])
    assert np.all(np.abs(got[:64] - want) <= 2e-7 * want + 1e-6), np.abs(got[:64] - want).max()
    if len(P) > 64:  # the last matrices of a batch, beyond one pass of the grid
        want = oracle.haralick_mcc(P[-64:])
        assert np.all(np.abs(got[-64:] - want) <= 2e-7 * want + 1e-6)
