"""A plan's partials of the level-slice kernel never move: a captured graph
stays right whatever eager calls come between its replays, and no call after
the creation (or, for plans the library makes itself, after the first) takes
more device memory."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1710_06189_amd as G  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu


def host(t):
    return t.view(torch.int32).cpu().numpy().view(np.uint32)


def dev(a):
    return torch.from_numpy(a).cuda()


# lo of the captured call and of the eager one: by level and by value in either order
@pytest.mark.parametrize("N,first,second", [(256, 0, 56), (256, 60, 0), (300, 0, 0), (300, 20, 10)])
@pytest.mark.parametrize("own", [True, False])
def test_replay_after_a_larger_eager_call(N, first, second, own):
    offs = [(1, 0), (-1, 1)]
    H, W = 900, 1300
    small, large = synth.smooth(200, 300, 3.0, 1), synth.uniform(H, W, 2)
    plan = G.glcm_plan_create(np.uint8, N, offs, W, H) if own else None
    t, big = dev(small), dev(large)
    out = torch.zeros((2, N, N), dtype=torch.int32, device="cuda").view(torch.uint32)
    side = torch.cuda.Stream()
    try:
        G.glcm_compute(t, N, first, 255, offs, out=out, plan=plan)  # (plan = None: its plan and partials)
        held = G.glcm_plan_workspace(plan) if own else G.glcm_plan_cache_stats()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            G.glcm_compute(t, N, first, 255, offs, out=out, plan=plan, stream=side)
        for rep in range(3):
            eager = host(G.glcm_compute(big, N, second, 255, offs, plan=plan))
            assert np.array_equal(eager, oracle.glcm(large, N, second, 255, offs))
            assert (G.glcm_plan_workspace(plan) if own else G.glcm_plan_cache_stats()) == held
            new = synth.smooth(200, 300, 3.0, 20 + rep)
            t.copy_(dev(new))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(host(out), oracle.glcm(new, N, first, 255, offs))
    finally:
        torch.cuda.synchronize()
        if own:
            plan.close()
