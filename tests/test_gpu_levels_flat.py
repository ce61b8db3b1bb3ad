"""Flat images at large N, bit for bit, where the level-slice kernel adds a
lane's pairs at once: rows that end anywhere in a wavefront, bands of one step,
flat parts beside noise, and the allocation-free entry point with all of its
memory as partials."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu

OFFS = [(1, 0), (-3, 2), (0, 1)]


def host(t):
    return t.view(torch.int32).cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("W", [15, 16, 17, 31, 100, 300, 1023, 1024, 1025, 2100])
@pytest.mark.parametrize("dtype,N", [(np.uint8, 256), (np.uint8, 300), (np.uint16, 400)])
def test_flat_rows(W, dtype, N):
    H, top = 260, int(np.iinfo(dtype).max)
    img = np.full((H, W), top // 3, dtype=dtype)
    img[90:140] = synth.uniform(50, W, W, dtype)  # flat, noise, flat and a step inside the rows
    img[200:, W // 2:] = top
    t = torch.from_numpy(img.view(np.int16)).cuda().view(torch.uint16) if dtype == np.uint16 else torch.from_numpy(img).cuda()
    want = oracle.glcm(img, N, 0, top, OFFS)
    assert np.array_equal(host(G.glcm_compute(t, N, 0, top, OFFS)), want)
    if 3 * N * N <= G.STATIC_MAX_WORDS:
        assert np.array_equal(host(G.glcm_compute_static(t, N, 0, top, OFFS)), want)


@pytest.mark.parametrize("N,K", [(256, 1), (256, 4), (200, 2), (512, 1)])
def test_static_fills_its_memory(N, K):
    """One offset's slices are an eighth of the static array's part; the bands
    of a large image take the rest of it."""
    img = synth.uniform(1100, 2300, N + K)
    t, offs = torch.from_numpy(img).cuda(), OFFS[:K] + [(2, 2)][:max(0, K - 3)]
    want = oracle.glcm(img, N, 0, 255, offs)
    for _ in range(2):
        assert np.array_equal(host(G.glcm_compute_static(t, N, 0, 255, offs)), want)
