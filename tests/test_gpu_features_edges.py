"""The five statistics at the edges of their kernels (whole rows per wavefront
step, 64-column blocks, 1, 4 and 16 wavefronts a matrix) against the oracle,
and batches against single calls bit for bit where a batch takes the matrix
that a workgroup takes alone."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402

pytestmark = pytest.mark.gpu


def counts(K, N, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    P = g.integers(0, 900, size=(K, N, N)).astype(np.uint32)
    P[g.random((K, N, N)) > 0.6] = 0
    P[K // 2] = 0
    P[0, N - 1, 0] = 3_000_000_000 if N > 1 else 7  # a bin above half of the total (the total below 2^32)
    return P


@pytest.mark.parametrize("N", [1, 2, 3, 7, 16, 21, 22, 31, 32, 33, 43, 63, 64, 65, 100, 127, 128, 129, 200, 256, 300, 1024])
def test_features_edges(N):
    """1e-5 relative, as the library states; exact zeros come out as zeros."""
    P = counts(5, N, N)
    got = G.glcm_features(torch.from_numpy(P.view(np.int32)).cuda()).cpu().numpy().astype(np.float64)
    want = oracle.features(P)
    assert np.all(got[want == 0] == 0)
    assert np.all(np.abs(got - want) <= 1e-5 * np.abs(want) + 1e-7 * (np.arange(5) == 4)), np.abs(got - want).max()


def test_totals_beyond_32_bits_are_nan():
    for N in (8, 40, 200):
        P = np.full((1, N, N), 2 ** 32 - 1, dtype=np.uint32)
        assert np.isnan(G.glcm_features(torch.from_numpy(P.view(np.int32)).cuda()).cpu().numpy()).all()


@pytest.mark.parametrize("N,K", [(31, 4), (33, 4), (43, 4), (60, 2), (85, 1)])
def test_batch_features_equal_single_calls(N, K):
    offs = [(1, 0), (0, 1), (1, 1), (-1, 1)][:K]
    g = np.random.Generator(np.random.PCG64(N))
    tiles = [torch.from_numpy(g.integers(0, 256, size=s, dtype=np.uint8)).cuda() for s in ((40, 71), (97, 33), (128, 128))]
    plan = G.glcm_plan_create(np.uint8, N, offs, 256, 256)
    try:
        P, F = G.glcm_batch_compute(tiles, plan)
        for t, tile in enumerate(tiles):
            one = G.glcm_compute(tile, N, 0, 255, offs)
            assert torch.equal(one.view(torch.int32), P[t].view(torch.int32))
            assert torch.equal(G.glcm_features(one).view(torch.int32), F[t].view(torch.int32))
    finally:
        plan.close()
