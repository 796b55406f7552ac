"""Instances of more than 64 segments of obstacles, whose lists a stage walks one after
the other: lists that hold nearly every obstacle, a few of the first or of the last
segments, or none of the first 64; open chains; all edge classes."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2607_04310_amd import inputs
from test_gpu_cull import _big, _chain_map

pytestmark = pytest.mark.gpu


def _rects(rng, M, half, order):
    e = inputs.random_rects(rng, M, 0.1, 0.8, -half, half).reshape(M, 16)
    far = np.hypot(e[:, 0], e[:, 1])
    key = {"mixed": rng.random(M), "near first": far, "near last": -far}[order]
    return e[np.argsort(key)].reshape(-1, 4), inputs.csr_offsets([4] * M)


def _same(insts, mbar, params=None):
    import torch
    from paper_2607_04310_amd import api
    a = api.Batch(insts, mbar=mbar, params=params)
    b = api.Batch(insts, mbar=mbar, params=params, graph=False, exhaustive=True)
    for _ in range(2):
        for name, x, y in zip(("d", "edge", "obst", "grad", "keys"), a.run(), b.run()):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name
    a.close()
    b.close()


@pytest.mark.parametrize("order", ["mixed", "near first", "near last"])
@pytest.mark.parametrize("M", [65536, 65537, 140000])
def test_rectangles(M, order):
    rng = np.random.default_rng([15, M])
    half = 40 * np.sqrt(M / 16384)
    e, off = _rects(rng, M, half, order)
    insts = [_big(rng, inputs.hexagon_footprint(rng))]
    for N, spread in ((70, 3.0), (60, half), (1, 1.0)):
        insts.append(SimpleNamespace(footprint=inputs.rect_footprint(), edges=e, obst_off=off,
                                     poses=inputs.uniform_poses(rng, N, -spread, spread)))
    _same(insts, 4)


@pytest.mark.parametrize("mbar,N", [(4, 150), (8, 150), (16, 150)])
def test_chains_and_polygons(mbar, N):
    rng = np.random.default_rng([16, mbar])
    M = 70000
    if mbar == 4:
        e, off = _chain_map(rng, M, 80.0, "chains")
    else:
        c, a = rng.uniform(-80, 80, (M, 1, 2)), np.arange(mbar) * 2 * np.pi / mbar
        P = c + rng.uniform(0.1, 0.6, (M, 1, 1)) * np.stack([np.cos(a), np.sin(a)], 1)
        e = np.concatenate([P, np.roll(P, -1, 1)], 2).reshape(-1, 4).astype(np.float32)
        off = inputs.csr_offsets([mbar] * M)
    fp = np.array([[-0.5, 0.0], [0.5, -0.176], [0.5, 0.176]], np.float32)
    poses = inputs.uniform_poses(rng, N, -80, 80)
    poses[3, 0], poses[5, 2] = np.nan, np.inf
    _same([SimpleNamespace(footprint=fp, poses=poses, edges=e, obst_off=off)], mbar)
