"""Post-processing at the edges of its kernels: matrices held by a wavefront
(N <= 16, N <= 32) and by workgroups (N > 32, split over several), bases off
the 16-byte grid, more matrices than the grid has wavefronts, totals beyond 32
bits.  Symmetric, normalised and averaged matrices bit for bit, Haralick's
statistics within 1e-5 relative (plus 1e-6 absolute on f3, f12 and f13, which
are cancellations near zero)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402

pytestmark = pytest.mark.gpu


def counts(K, N, seed, high=5000, density=0.7):
    g = np.random.Generator(np.random.PCG64(seed))
    P = g.integers(0, high, size=(K, N, N), dtype=np.uint64).astype(np.uint32)
    P[g.random((K, N, N)) > density] = 0
    P[K // 2] = 0
    return P


def dev(P, shift=0):
    """P on the GPU, its base `shift` words past an aligned one."""
    flat = torch.zeros(P.size + shift, dtype=torch.int32, device="cuda")
    flat[shift:] = torch.from_numpy(P.view(np.int32).reshape(-1)).cuda()
    return flat[shift:].view(P.shape).view(torch.uint32)


def host(t):
    return t.cpu().numpy() if t.dtype == torch.float32 else t.view(torch.int32).cpu().numpy().view(np.uint32)


def check(P, m, shift=0):
    t = dev(P, shift)
    sym = oracle.symmetric(P)
    assert np.array_equal(host(G.glcm_symmetrize(t)), sym)
    inplace = dev(P, shift)
    G.glcm_symmetrize(inplace, out=inplace)
    assert np.array_equal(host(inplace), sym)
    assert np.array_equal(host(G.glcm_normalize(t)), oracle.normalize(P).astype(np.float32))
    assert np.array_equal(host(G.glcm_average(t, m)), oracle.average(P, m).astype(np.float32))
    if P.shape[1] <= 1024:
        got, want = host(G.glcm_haralick(t)).astype(np.float64), oracle.haralick(P)
        tol = 1e-5 * np.abs(want)
        tol[:, [2, 11, 12]] += 1e-6
        bad = np.abs(got - want) > tol
        assert not bad.any(), (np.argwhere(bad)[:5], got[bad][:5], want[bad][:5])


@pytest.mark.parametrize("N", [1, 2, 3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 127, 255, 256, 257, 300])
@pytest.mark.parametrize("shift", [0, 1])
def test_edges(N, shift):
    check(counts(6, N, 100 + N), 3, shift)


@pytest.mark.parametrize("K,N,m,high", [
    (4099, 5, 1, 300),          # one more group than the grid's wavefronts hold at once
    (9001, 3, 9001 // 9001, 50),
    (8448, 4, 64, 50),          # the largest group
    (300, 70, 4, 9),            # more matrices than CUs above 32 levels
    (4, 1000, 2, 40),           # few large ones, split over the chip
    (3, 12, 3, 2 ** 32), (3, 30, 3, 2 ** 32), (3, 100, 3, 2 ** 32),  # totals beyond 32 bits
])
def test_many_and_large(K, N, m, high):
    check(counts(K, N, K + N, high), m)


def test_unused_levels_and_single_bins():
    """Statistics of matrices with one occupied bin or diagonal: exact zeros."""
    for N in (16, 24, 40):
        P = np.zeros((4, N, N), dtype=np.uint32)
        P[0, 3, N - 2] = 99
        P[1][np.arange(N), np.arange(N)] = 3
        P[2, :, 5] = np.arange(1, N + 1)
        P[3, N - 1, N - 1] = 2 ** 32 - 1
        check(P, 2)
        got = host(G.glcm_haralick(dev(P)))
        assert got[2, 2] == 1.0 and got[0, 8] == 0.0 and got[1, 1] == 0.0
