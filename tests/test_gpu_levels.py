"""The level-slice kernel (large N) against the oracle, bit for bit: one and
several slices, bins emptied before they overflow (constant and two-level
images), rectangles narrower than a 16-pixel load, any alignment, offsets
leaving the image, host images in tiles, the allocation-free entry point and a
captured first call."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu

ALL12 = synth.offsets_for([1, 2, 4])


def dev(a):
    return torch.from_numpy(a.view(np.int16)).cuda().view(torch.uint16) if a.dtype == np.uint16 else torch.from_numpy(a).cuda()


def host(t):
    return t.view(torch.int32).cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("H,W,dtype,N,offs,lo,hi", [
    (300, 400, np.uint8, 256, ALL12, 0, 255),
    (257, 1031, np.uint8, 256, [(-3, 2), (5, -7), (0, -4), (-16, 0)], 0, 255),
    (90, 70, np.uint8, 200, [(60, 1), (-58, 3), (69, 0), (70, 0), (0, 90), (1, 89)] + ALL12[:3], 20, 230),
    (40, 9, np.uint8, 256, [(1, 0), (-8, 5), (0, 1)], 0, 255),          # rows narrower than a load
    (1, 5000, np.uint8, 256, [(1, 0), (0, 1)], 0, 255),
    (5000, 1, np.uint8, 256, [(0, 1), (1, 1)], 0, 255),
    (333, 517, np.uint16, 256, ALL12[:5], 0, 65535),
    (200, 333, np.uint16, 300, [(1, 0), (-2, 2), (0, -3), (7, 7)], 100, 60000),
    (150, 700, np.uint16, 1000, [(1, 0), (2, 2)], 0, 65535),             # several slices
    (64, 2000, np.uint8, 1024, [(1, 0), (-1, 1)], 0, 255),               # more levels than values
    (300, 300, np.uint8, 65, [(20, 0), (0, 20)] * 6, 0, 255),            # small matrices, offsets beyond the row kernels
])
@pytest.mark.parametrize("shift", [0, 3])
def test_levels(H, W, dtype, N, offs, lo, hi, shift):
    top = int(np.iinfo(dtype).max)
    base = synth.smooth(H + 2, W + 8, 3.0, H + W, dtype) if min(H, W) > 8 else synth.uniform(H + 2, W + 8, H + W, dtype)
    noise = synth.uniform(H + 2, W + 8, H + W + 1, dtype)
    plan = G.glcm_plan_create(dtype, N, offs, W, H)
    try:
        for img in (base, noise, np.full_like(base, top // 3)):
            view = dev(img)[1:1 + H, shift:shift + W]
            got = host(G.glcm_compute(view, N, lo, hi, offs, plan=plan))
            assert np.array_equal(got, oracle.glcm(img[1:1 + H, shift:shift + W], N, lo, hi, offs))
    finally:
        plan.close()


@pytest.mark.parametrize("kind", ["constant", "two levels", "half and half"])
@pytest.mark.parametrize("N,offs", [(256, [(1, 0), (0, 1), (-1, 1)]), (512, [(0, 1)])])
def test_bins_that_overflow(kind, N, offs):
    """Millions of pairs in one, two or a few bins: every 16-bit bin is
    emptied many times."""
    H, W = 2500, 3000
    img = np.full((H, W), 77, dtype=np.uint8)
    if kind == "two levels":
        img[:, ::2] = 200
    elif kind == "half and half":
        img[:, 1000:] = synth.uniform(H, W - 1000, 5)
    got = host(G.glcm_compute(dev(img), N, 0, 255, offs))
    assert np.array_equal(got, oracle.glcm(img, N, 0, 255, offs))


def test_host_tiles_and_static():
    img = synth.smooth(700, 900, 4.0, 8)
    want = oracle.glcm(img, 256, 0, 255, ALL12[:4])
    plan = G.glcm_plan_create(np.uint8, 256, ALL12[:4], 900, 700)
    try:
        plan.set_tuning(tile_rows=100)
        for _ in range(2):
            assert np.array_equal(host(G.glcm_compute(img, 256, 0, 255, ALL12[:4], plan=plan)), want)
        assert np.array_equal(host(G.glcm_compute(dev(img), 256, 0, 255, ALL12[:4], plan=plan)), want)
    finally:
        plan.close()
    for _ in range(2):
        assert np.array_equal(host(G.glcm_compute_static(dev(img), 256, 0, 255, ALL12[:4])), want)
    one = synth.uniform(3000, 2000, 4)
    assert np.array_equal(host(G.glcm_compute_static(dev(one), 500, 0, 255, [(1, 1)])), oracle.glcm(one, 500, 0, 255, [(1, 1)]))


def test_first_call_under_capture():
    """A rebound plan whose partials were never needed: its first call under
    capture may not allocate, takes the ranges of 32-bit bins, and replays."""
    near, far = ALL12, [(9 + k, k) for k in range(12)]
    img = synth.smooth(200, 300, 3.0, 9)
    t = dev(img)
    plan = G.glcm_plan_create(np.uint8, 100, near, 300, 200)
    out = torch.zeros((12, 100, 100), dtype=torch.int32, device="cuda").view(torch.uint32)
    side = torch.cuda.Stream()
    try:
        G.glcm_plan_rebind(plan, far)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            G.glcm_compute(t, 100, 0, 255, far, out=out, plan=plan, stream=side)
        for rep in range(3):
            new = synth.smooth(200, 300, 3.0, 20 + rep)
            t.copy_(dev(new))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(host(out), oracle.glcm(new, 100, 0, 255, far))
    finally:
        torch.cuda.synchronize()
        plan.close()


@pytest.mark.parametrize("dtype,N,lo,hi", [
    (np.uint8, 257, 0, 255), (np.uint8, 300, 0, 255), (np.uint8, 1024, 0, 255), (np.uint8, 1000, 60, 255),
    (np.uint8, 1000, 20, 230),           # pixels above hi: level N - 1, which no value has
    (np.uint16, 400, 65300, 65535),      # a window of a 16-bit image
    (np.uint16, 300, 65236, 65535),      # more values than one slice holds
])
def test_fewer_values_than_levels(dtype, N, lo, hi):
    top = int(np.iinfo(dtype).max)
    img = synth.uniform(300, 700, N + lo, np.uint8).astype(dtype) + dtype(top - 255)
    img[:150] = top // 2 if dtype == np.uint8 else top - 100
    img[:40, :200] = 0
    offs = [(1, 0), (-1, 1), (0, 2)]
    got = host(G.glcm_compute(dev(img), N, lo, hi, offs))
    assert np.array_equal(got, oracle.glcm(img, N, lo, hi, offs))
    big = np.tile(img, (8, 3))  # the bins of the constant part overflow and spill
    assert np.array_equal(host(G.glcm_compute(dev(big), N, lo, hi, offs)), oracle.glcm(big, N, lo, hi, offs))
