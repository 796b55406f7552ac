"""The bound form where eps leaves the circles no bound: every pair is evaluated, as
psdf_batch does, eager, from staged edges and in a captured graph whose replays see
changed poses."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2607_04310_amd import inputs
from test_gpu_cull import ODD, _inst

pytestmark = pytest.mark.gpu


def _same(got, want):
    import torch
    return all(torch.equal(g.view(torch.uint8), w.view(torch.uint8)) for g, w in zip(got, want))


@pytest.mark.parametrize("eps", [2e-6, 1e-2])
def test_bound_form_equals_the_batch(eps):
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(17)
    fps = [inputs.rect_footprint(), inputs.hexagon_footprint(rng), inputs.random_convex_footprint(rng, 3),
           inputs.random_convex_footprint(rng, 8)]
    insts = [_inst(rng, fp, N, M, 12.0, odd=ODD) for fp in fps for N, M in ((20, 900), (3, 40))]
    insts.append(SimpleNamespace(footprint=fps[0], poses=inputs.path_poses(rng, 5, -1, 1),
                                 edges=np.zeros((0, 4), np.float32), obst_off=np.zeros(1, np.int32)))
    pr = api.Params(eps=eps)
    a = api.Batch(insts, mbar=4, params=pr, graph=False)
    b = api.Batch(insts, mbar=4, params=pr, graph=False, exhaustive=True)
    assert _same(a.screened_bound(), b.run())
    assert _same(a.stage().screened_bound(), b.run())
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            a.screened_bound()
    torch.cuda.synchronize()
    for k in range(3):
        move = torch.tensor(rng.normal(0, 0.3, tuple(a.poses.shape)).astype(np.float32), device="cuda")
        a.poses += move
        b.poses += move
        for t in (a.d, a.edge, a.obst, a.grad, a.keys):
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert _same((a.d, a.edge, a.obst, a.grad, a.keys), b.run()), k
        assert _same(a.screened_bound(), b.run()), k
    a.close()
    b.close()
