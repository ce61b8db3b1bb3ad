"""Up to 16 levels on the matrix cores, bit for bit against the oracle: widths
and heights around its windows and row blocks, every reach, negated and
repeated offsets, pixels at any alignment, counts near what its sums hold,
host tiles, one workgroup and many, batches with bands."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu

ALL12 = synth.offsets_for([1, 2, 4])
D1, D2 = ALL12[:4], ALL12[:8]
SETS = {
    "one": [(1, 0)], "d1": D1, "d1 negated": [(-1, 0), (1, -1), (0, -1), (-1, -1), (1, 0), (1, 0)],
    "d2": D2, "some of d2": [(2, 0), (-2, 2), (0, -2), (-2, -2), (0, 1)], "d4": ALL12,
    "some of d4": [(4, 0), (4, -4), (0, 4), (-1, 1), (-4, -4)],
}


def dev(a):
    return torch.from_numpy(a.view(np.int16)).cuda().view(torch.uint16) if a.dtype == np.uint16 else torch.from_numpy(a).cuda()


def host(t):
    return t.view(torch.int32).cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("name", list(SETS))
@pytest.mark.parametrize("W,H", [(1, 1), (5, 3), (31, 17), (32, 16), (33, 15), (62, 1), (63, 2), (64, 64), (92, 31), (93, 46),
                                 (120, 33), (200, 300), (1000, 90), (1031, 500)])
def test_sizes(name, W, H):
    offs = SETS[name]
    for dtype, N, lo, hi in ((np.uint8, 16, 0, 255), (np.uint16, 8, 0, 65535), (np.uint8, 13, 30, 200), (np.uint16, 3, 500, 60000)):
        base = synth.uniform(H + 1, W + 6, W + H, dtype)
        base[H // 2:, W // 3:] = base[0, 0]
        view = dev(base)[1:, 3:3 + W]
        got = host(G.glcm_compute(view, N, lo, hi, offs))
        assert np.array_equal(got, oracle.glcm(base[1:, 3:3 + W], N, lo, hi, offs)), (dtype, N)


@pytest.mark.parametrize("N", list(range(1, 18)))
def test_levels(N):
    img = synth.smooth(130, 170, 2.0, N)
    for offs in (D1, D2, ALL12):
        assert np.array_equal(host(G.glcm_compute(dev(img), N, 0, 255, offs)), oracle.glcm(img, N, 0, 255, offs))


@pytest.mark.parametrize("kind", ["constant", "noise", "smooth"])
@pytest.mark.parametrize("offs", [D1, ALL12], ids=["d1", "d4"])
def test_large(kind, offs):
    H, W = 4096, 4100
    img = {"constant": lambda: np.full((H, W), 130, np.uint8), "noise": lambda: synth.uniform(H, W, 3),
           "smooth": lambda: synth.smooth(H, W, 8.0, 4)}[kind]()
    assert np.array_equal(host(G.glcm_compute(dev(img), 16, 0, 255, offs)), oracle.glcm(img, 16, 0, 255, offs))


def test_tall_wide_and_host_tiles():
    for shape in ((60000, 37), (3, 65000), (20000, 640)):
        img = synth.uniform(*shape, 6)
        assert np.array_equal(host(G.glcm_compute(dev(img), 16, 0, 255, D2)), oracle.glcm(img, 16, 0, 255, D2))
    img = synth.smooth(500, 700, 3.0, 8)
    for offs in (D1, ALL12, SETS["some of d4"]):
        plan = G.glcm_plan_create(np.uint8, 16, offs, 700, 500)
        try:
            for rows in (1, 2, 40, 499):
                plan.set_tuning(tile_rows=rows)
                assert np.array_equal(host(G.glcm_compute(img, 16, 0, 255, offs, plan=plan)), oracle.glcm(img, 16, 0, 255, offs)), rows
            assert np.array_equal(host(G.glcm_compute(dev(img), 16, 0, 255, offs, plan=plan)), oracle.glcm(img, 16, 0, 255, offs))
        finally:
            plan.close()
    for small in (img[:40, :50], img):
        t = dev(np.ascontiguousarray(small))
        for _ in range(2):
            assert np.array_equal(host(G.glcm_compute_static(t, 16, 0, 255, D1)), oracle.glcm(small, 16, 0, 255, D1))


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("name,N", [("d1", 16), ("d1", 5), ("some of d2", 16)])
def test_batches(dtype, name, N):
    """Small, narrow, tall and split images, rows at any alignment; statistics
    equal those of single calls bit for bit, and of the LDS kernel."""
    offs, top = SETS[name][:4], int(np.iinfo(dtype).max)
    shapes = [(1, 1), (2, 40), (33, 7), (64, 64), (17, 31), (16, 33), (100, 515), (512, 512), (1500, 900), (3, 3000), (5000, 260)]
    big = synth.smooth(5001, 3003, 3.0, 11, dtype)
    big[:700] = synth.uniform(700, 3003, 12, dtype)
    views = [dev(big)[y % 7:y % 7 + h, 1 + y:1 + y + w] for y, (h, w) in enumerate(shapes)]
    plan = G.glcm_plan_create(dtype, N, offs, 3000, 5000)
    try:
        P, F = G.glcm_batch_compute(views, plan, 0, top)
        batch = G.PreparedBatch(views, plan)
        for _ in range(3):
            P2, F2 = batch.run(0, top, features=True)
            assert torch.equal(P.view(torch.int32), P2.view(torch.int32)) and torch.equal(F.view(torch.int32), F2.view(torch.int32))
        for y, (h, w) in enumerate(shapes):
            want = oracle.glcm(big[y % 7:y % 7 + h, 1 + y:1 + y + w], N, 0, top, offs)
            assert np.array_equal(host(P)[y], want), (h, w)
            assert torch.equal(G.glcm_features(P[y]).view(torch.int32), F[y].view(torch.int32))
        plan.set_batch_tuning(replicas=8)
        P3, F3 = G.glcm_batch_compute(views, plan, 0, top)
        assert torch.equal(P.view(torch.int32), P3.view(torch.int32)) and torch.equal(F.view(torch.int32), F3.view(torch.int32))
    finally:
        torch.cuda.synchronize()
        plan.close()


@pytest.mark.parametrize("name,N", [("d1", 16), ("some of d2", 7)])
def test_many_images(name, N):
    """More images than workgroups: the small ones are counted by a wavefront
    each, next to large ones, 2^13 pixels (the line between them) on both
    sides; the LDS kernel gives the same bits."""
    offs = SETS[name][:4]
    big = synth.smooth(700, 801, 3.0, 13, np.uint8)
    g = np.random.default_rng(14)
    shapes = [(1, 1), (64, 127), (64, 128), (64, 129), (128, 64), (300, 310), (600, 790), (1, 60), (60, 1)]
    shapes += [tuple(int(v) for v in g.integers(1, 100, 2)) for _ in range(1291)]
    src = dev(big)
    views = [src[y % 50:y % 50 + h, y % 11:y % 11 + w] for y, (h, w) in enumerate(shapes)]
    plan = G.glcm_plan_create(np.uint8, N, offs, 801, 700)
    try:
        batch = G.PreparedBatch(views, plan)
        for _ in range(3):
            P, F = batch.run(20, 230, features=True)
        for y in [*range(9), *range(9, 1300, 97)]:
            h, w = shapes[y]
            assert np.array_equal(host(P[y]), oracle.glcm(big[y % 50:y % 50 + h, y % 11:y % 11 + w], N, 20, 230, offs)), (h, w)
        plan.set_batch_tuning(replicas=8)
        P2, F2 = G.glcm_batch_compute(views, plan, 20, 230)
        assert torch.equal(P.view(torch.int32), P2.view(torch.int32)) and torch.equal(F.view(torch.int32), F2.view(torch.int32))
    finally:
        torch.cuda.synchronize()
        plan.close()


@pytest.mark.parametrize("W", [1 << 19, (1 << 19) + 1])
def test_widest_images(W):
    """Images too wide for the matrix cores' sums go to the LDS kernel."""
    img = synth.uniform(2, W, 15, np.uint8)
    plan = G.glcm_plan_create(np.uint8, 16, D1, W, 2)
    try:
        P, _ = G.glcm_batch_compute([dev(img), dev(img)], plan, 0, 255)
        assert np.array_equal(host(P[1]), oracle.glcm(img, 16, 0, 255, D1))
    finally:
        torch.cuda.synchronize()
        plan.close()
