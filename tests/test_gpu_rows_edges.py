"""The whole-row kernel bit for bit against the oracle where its spans of 1024
pixels and its runs of rows end: widths around a span, a chunk and the halos,
heights from one row to more than a workgroup's runs, aligned and unaligned rows."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu

SETS = {
    1: [(1, 0), (1, -1), (0, -1), (-1, -1), (-1, 1)],
    2: [(2, 0), (-2, 1), (0, -2), (2, 2), (-1, -1), (-2, -2)],
    4: [(4, 0), (-4, 0), (4, 4), (-4, 4), (0, -4), (3, 1), (-3, 2), (1, 3), (-2, -4), (2, -3)],
}


@pytest.mark.parametrize("reach", [1, 2, 4])
@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("W", [1, 4, 15, 17, 1020, 1021, 1024, 1025, 1029, 2047, 2051])
def test_edges(reach, dtype, W):
    top, offs = int(np.iinfo(dtype).max), SETS[reach]
    img = synth.uniform(601, W + 32, 17 + W, dtype)
    dev = torch.from_numpy(img.view(np.int16) if dtype == np.uint16 else img).cuda()
    dev = dev.view(torch.uint16) if dtype == np.uint16 else dev
    for H, x in ((1, 0), (2, 0), (5, 1), (33, 0), (600, 0), (601, 3)):
        plan = G.glcm_plan_create(dtype, 40, offs, W, H, G.FLAG_FORCE_SLABS)
        try:
            got = G.glcm_compute(dev[:H, x:x + W], 40, 0, top, offs, plan=plan)
            want = oracle.glcm(img[:H, x:x + W], 40, 0, top, offs)
            assert np.array_equal(got.view(torch.int32).cpu().numpy().view(np.uint32), want), (H, x)
        finally:
            plan.close()
