"""Geometry adjoint of winners of one to four edges, whose pool pairs are a lane
each and read the footprint's table across the wave: one-stage calls with
footprints of 3 to 16 vertices in turn (each call finds the previous one's table
in LDS), against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2607_04310_amd import inputs

pytestmark = pytest.mark.gpu

G_RTOL = 1e-4   # the repository's gradient tolerance


@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_few_edges_every_footprint_size(k):
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng([3, k])
    one = torch.ones(1, device="cuda")
    for m in (16, 3, 12, 5, 8, 4, 7, 6, 9, 16):
        ang = 2 * np.pi * (np.arange(m) + rng.uniform(-0.2, 0.2, m)) / m
        fp = np.stack([0.5 * np.cos(ang), 0.35 * np.sin(ang)], 1).astype(np.float32)
        a = np.sort(rng.uniform(0, 2 * np.pi, k)) if k > 2 else rng.uniform(0, 2 * np.pi, k + 1)
        P = (rng.uniform(0.9, 2.0) + 0.4 * np.stack([np.cos(a), np.sin(a)], 1)).astype(np.float32)
        edges = np.concatenate([P, np.roll(P, -1, 0)] if k > 2 else [P[:-1], P[1:]], 1)
        pose = np.array([[0.1, -0.05, rng.uniform(-3, 3)]], np.float32)
        es = api.EdgeSet(edges, inputs.csr_offsets([k]), 4)
        x = torch.tensor(pose, device="cuda")
        keys = api.psdf_grad(fp, x, es)[4]
        gE, gF = (t.cpu().numpy() for t in api.psdf_bwd_geometry(fp, x, es, keys, one))
        ge, gf = oracle.geom_grad(fp, pose[0], edges)
        tol = G_RTOL * max(1.0, np.abs(ge).max(), np.abs(gf).max())
        assert np.abs(gF - gf).max() <= tol, (m, gF, gf)
        total = lambda G: G[:, :2].sum(0) + G[:, 2:].sum(0)
        assert np.abs(total(gE) - total(ge)).max() <= tol, (m, gE, ge)
