"""The culled evaluation far from the map's origin, where the boxes' own
rounding is centimetres to decimetres, with footprints that lie ahead of the
pose origin (a trailer, a tool): outputs equal the full evaluation's bit for
bit, also where two obstacles on opposite sides differ by less than that
rounding."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2607_04310_amd import inputs

pytestmark = pytest.mark.gpu


def _pairs(rng, n, at, span):
    """n instances of one stage: a footprint c metres ahead of its origin, a
    segment behind it that ends near the pose and a short one beyond it, at about
    the same distance on the float grid around `at`."""
    out = []
    for k in range(n):
        c, h = rng.uniform(1.0, 8.0), rng.uniform(0.02, 0.3)
        if k == 0:
            c, h = 3.027, 0.02
        fp = np.array([[c - h, -h], [c + h, -h], [c + h, h], [c - h, h]], np.float32)
        p = np.array([at if k == 0 else at + rng.uniform(-1000, 1000), 0.0], np.float32)
        xi = np.float32(p[0] + (-8.0 if k == 0 else c - h - rng.uniform(1.0, span)))
        gap = float(p[0]) + c - h - float(xi)
        xj = np.float32(float(p[0]) + c + h + gap - rng.uniform(0.0, 0.2))
        if k == 0:
            xj = np.float32(at + 14.0)
        seg = np.array([[xi - 5.0, 0.0, xi, 0.0], [xj, -0.01, xj, 0.01]], np.float32)
        out.append(SimpleNamespace(footprint=fp, poses=np.array([[p[0], p[1], 0.0]], np.float32),
                                   edges=seg[::-1].copy() if k % 2 else seg,
                                   obst_off=inputs.csr_offsets([1, 1])))
    return out


@pytest.mark.parametrize("at,span", [(624950.0, 20.0), (5.0e6, 60.0), (-3.0e4, 20.0)])
def test_far_from_the_origin(at, span):
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(7)
    big = SimpleNamespace(footprint=inputs.rect_footprint(), poses=inputs.path_poses(rng, 300, -20, 20),
                          edges=inputs.random_rects(rng, 16384, 0.1, 0.8, -20, 20),
                          obst_off=inputs.csr_offsets([4] * 16384))
    insts = [big] + _pairs(rng, 8000, at, span)
    a = api.Batch(insts, mbar=4)
    want = [t.clone() for t in api.Batch(insts, mbar=4, graph=False, exhaustive=True).run()]
    for form, call in (("culled", a.run), ("bound", a.screened_bound),
                       ("bound, staged", lambda: a.stage().screened_bound())):
        got = [t.clone() for t in call()]
        torch.cuda.synchronize()
        for name, g, w in zip(("d", "edge", "obst", "grad", "keys"), got, want):
            g, w = g.cpu().numpy(), w.cpu().numpy()
            bad = np.flatnonzero((g.view(np.uint8) != w.view(np.uint8)).reshape(len(g), -1).any(1))
            assert len(bad) == 0, (form, name, len(bad), bad[:5], g[bad[:5]], w[bad[:5]])
