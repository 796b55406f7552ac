"""Needles of a footprint where the culled forms are taken (the routes of these sizes
are in test_host_plans.py): a batch whose needles meet at most one segment of
obstacles, also a needle without a bound, and plain calls large enough for them."""
import numpy as np
import pytest

from paper_2607_04310_amd import inputs
from test_gpu_cull import ODD, SLIVERS, _big, _check, _inst

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", range(len(SLIVERS)))
def test_needles_in_a_culled_batch(k):
    rng = np.random.default_rng([13, k])
    fp = SLIVERS[k]
    _check([_big(rng, inputs.rect_footprint()), _inst(rng, fp, 30, 1000, 15.0),
            _inst(rng, fp, 70, 900, 15.0, odd=ODD[:8]), _inst(rng, fp, 3, 5, 2.0, odd=ODD)])


@pytest.mark.parametrize("kind", ["rects", "mixed"])
@pytest.mark.parametrize("w", [0.1, 0.0437, 8.7e-4])
def test_needles_in_a_plain_call(kind, w):
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(14)
    fp = np.array([[-0.5, 0.0], [0.5, -w], [0.5, w]], np.float32)
    if kind == "rects":
        e, off = inputs.random_rects(rng, 30011, 0.1, 0.8, -60, 60), inputs.csr_offsets([4] * 30011)
    else:
        i = _inst(rng, fp, 1, 30011, 60.0, odd=ODD * 3)
        e, off = i.edges, i.obst_off
    es = api.EdgeSet(e, off, 4)
    poses = torch.tensor(inputs.uniform_poses(rng, 300, -60, 60)).cuda()
    a = api.psdf_grad(fp, poses, es)
    api.set_launch_shape(256, 8)
    try:
        b = api.psdf_grad(fp, poses, es)
    finally:
        api.set_launch_shape(0, 0)
    for name, x, y in zip(("d", "edge", "obst", "grad", "keys"), a, b):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name
