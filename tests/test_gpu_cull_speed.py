"""The evaluation that a call takes by itself is not the slower one on maps that
are not made of convex polygons, with footprints from blunt to needle: against
the full evaluation of every pair on the same inputs (the best of several
bursts of each), with the same outputs bit for bit."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2607_04310_amd import inputs

pytestmark = pytest.mark.gpu

HALF = 40.0       # 16384 obstacles of about a metre in 80 m x 80 m
FOOTPRINTS = {
    "hexagon": inputs.hexagon_footprint(np.random.default_rng(3)),
    "triangle": np.array([[0.5, 0.0], [-0.25, 0.433], [-0.25, -0.433]], np.float32),
    "20 degrees": np.array([[-0.5, 0.0], [0.5, -0.176], [0.5, 0.176]], np.float32),
    "5 degrees": np.array([[-0.5, 0.0], [0.5, -0.0437], [0.5, 0.0437]], np.float32),
    "0.1 degrees": np.array([[-0.5, 0.0], [0.5, -8.7e-4], [0.5, 8.7e-4]], np.float32),
}


def _closed(P):
    return np.concatenate([P, np.roll(P, -1, 1)], 2)


def _map(rng, M, kind):
    """(edges, offsets, mbar): `chains` of three edges, rectangles with a vertex
    within a side (`side`), `arrows` with a reflex corner."""
    c, a = rng.uniform(-HALF, HALF, (M, 1, 2)), rng.uniform(0, 2 * np.pi, M)
    R = np.stack([np.stack([np.cos(a), -np.sin(a)], 1), np.stack([np.sin(a), np.cos(a)], 1)], 1)
    w, h = rng.uniform(0.1, 0.8, (2, M, 1))
    z = 0 * w
    corner = lambda *xy: np.stack([np.concatenate(p, 1) for p in xy], 1) @ R.transpose(0, 2, 1) + c
    if kind == "chains":
        P = c + np.cumsum(rng.normal(0, 0.3, (M, 4, 2)), 1)
        e = np.concatenate([P[:, :-1], P[:, 1:]], 2)
    elif kind == "side":
        e = _closed(corner((-w, -h), (z, -h), (w, -h), (z, h)))
    else:
        e = _closed(corner((-w, -h), (z, -h / 3), (w, -h), (z, h)))
    return e.reshape(-1, 4).astype(np.float32), inputs.csr_offsets([e.shape[1]] * M), 4


def _time(torch, call, n=10):
    for _ in range(3):
        call()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / n)
    return best


def _batch(kind, fp, k=16, N=50, M=16384):
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(5)
    insts = []
    for _ in range(k):
        edges, off, mbar = _map(rng, M, kind)
        insts.append(SimpleNamespace(footprint=fp, poses=inputs.path_poses(rng, N, -HALF / 2, HALF / 2),
                                     edges=edges, obst_off=off))
    a = api.Batch(insts, mbar=mbar)
    b = api.Batch(insts, mbar=mbar, exhaustive=True)
    want = [t.clone() for t in b.run()]
    full = _time(torch, b.run)
    out = {}
    for form, call in (("culled", a.run), ("bound", a.screened_bound)):
        got = call()
        assert all(torch.equal(g.view(torch.uint8), w.view(torch.uint8)) for g, w in zip(got, want)), form
        out[form] = _time(torch, call)
    a.stage()
    got = a.screened_bound()
    assert all(torch.equal(g.view(torch.uint8), w.view(torch.uint8)) for g, w in zip(got, want))
    out["staged"] = _time(torch, a.screened_bound)
    a.close()
    b.close()
    print(kind, {k: round(1e3 * v, 1) for k, v in dict(full=full, **out).items()}, flush=True)
    return full, out


@pytest.mark.parametrize("kind", ["chains", "side", "arrows"])
@pytest.mark.parametrize("fp", ["hexagon", "triangle"])
def test_staging_does_not_slow_the_bound_form(kind, fp):
    """From staged boxes a call reads less; a tenth is left to noise."""
    full, out = _batch(kind, FOOTPRINTS[fp])
    assert out["staged"] <= 1.1 * out["bound"], (full, out)


@pytest.mark.parametrize("kind", ["chains", "side", "arrows"])
@pytest.mark.parametrize("fp", ["hexagon", "triangle", "20 degrees", "5 degrees"])
def test_batch_is_not_slower_than_the_full_evaluation(kind, fp):
    full, out = _batch(kind, FOOTPRINTS[fp])
    assert max(out.values()) <= 1.1 * full, (full, out)


@pytest.mark.parametrize("k,N,M", [(1, 300, 16384), (1, 2000, 16384), (1, 20000, 2048), (16, 100, 16384),
                                   (16, 200, 4096), (4, 200, 16384)])
@pytest.mark.parametrize("fp", ["20 degrees", "5 degrees", "0.1 degrees"])
def test_long_horizons_are_not_slower(fp, k, N, M):
    """(The bound form stays culled, and exact on chains, where the batch itself takes
    the full evaluation.)"""
    full, out = _batch("chains", FOOTPRINTS[fp], k, N, M)
    assert out["culled"] <= 1.25 * full, (full, out)


def _plain(fp, N, M, e, off, mbar):
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(7)
    es = api.EdgeSet(e, off, mbar)
    poses = torch.tensor(inputs.path_poses(rng, N, -HALF / 2, HALF / 2), device="cuda")
    blk, sb = (64 if M <= 1024 else 256), 1       # the full form's automatic shape
    while sb < 64 and (M + 63) // 64 * ((N + 2 * sb - 1) // (2 * sb)) >= 4096:
        sb *= 2
    ws = api.workspace(N, M, "cuda")
    res, ms = [], []
    for shape in ((0, 0), (blk, sb)):
        api.set_launch_shape(*shape)
        try:
            out = api.psdf_grad(fp, poses, es, ws=ws)
            res.append([t.clone() for t in out])
            ms.append(_time(torch, lambda: api.psdf_grad(fp, poses, es, out=out, ws=ws)))
        finally:
            api.set_launch_shape(0, 0)
    assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(*res))
    print(N, M, mbar, "chosen, full:", [round(1e3 * t, 1) for t in ms], flush=True)
    assert ms[0] <= 1.3 * ms[1], ms


@pytest.mark.parametrize("kind", ["chains", "side"])
@pytest.mark.parametrize("fp", FOOTPRINTS)
@pytest.mark.parametrize("N,M", [(100, 16384), (200, 16384), (200, 65536), (1000, 4096)])
def test_plain_call_is_not_slower(kind, fp, N, M):
    _plain(FOOTPRINTS[fp], N, M, *_map(np.random.default_rng(5), M, kind))


@pytest.mark.parametrize("m", [3, 4, 6, 16])
@pytest.mark.parametrize("mbar,M", [(8, 16), (8, 64), (8, 100), (8, 200), (16, 16), (4, 257), (4, 400)])
def test_many_stages_against_a_small_map(m, mbar, M):
    rng = np.random.default_rng(9)
    c = rng.uniform(-HALF / 8, HALF / 8, (M, 1, 2))
    a = np.arange(mbar) * 2 * np.pi / mbar + rng.uniform(0, 1, (M, 1))
    e = _closed(c + rng.uniform(0.1, 0.5, (M, 1, 1)) * np.stack([np.cos(a), np.sin(a)], 2))
    t = np.arange(m) * 2 * np.pi / m
    fp = (0.5 * np.stack([np.cos(t), np.sin(t)], 1)).astype(np.float32)
    _plain(fp, 20000, M, e.reshape(-1, 4).astype(np.float32), inputs.csr_offsets([mbar] * M), mbar)


def _octagons(rng, M, mbar, half):
    a = np.arange(mbar) * 2 * np.pi / mbar + rng.uniform(0, 1, (M, 1))
    e = _closed(rng.uniform(-half, half, (M, 1, 2)) +
                rng.uniform(0.1, 0.5, (M, 1, 1)) * np.stack([np.cos(a), np.sin(a)], 2))
    return e.reshape(-1, 4).astype(np.float32), inputs.csr_offsets([mbar] * M)


@pytest.mark.parametrize("mbar,k,N,M", [(4, 20, 1, 210000), (4, 3, 16, 130000), (4, 1, 32, 400000), (8, 257, 1, 16384),
                                        (16, 65, 2, 16384), (16, 65, 4, 16384), (4, 257, 1, 16384),
                                        (8, 2, 32, 130000), (16, 2, 32, 130000)])
def test_few_stages_per_instance(mbar, k, N, M):
    """Each obstacle is read for a stage or a few: batches of edge sets per stage, and
    instances of more than 64 segments."""
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(11)
    half = HALF * np.sqrt(M / 16384)
    maps = [_octagons(rng, M, mbar, half) for _ in range(2)]
    insts = [SimpleNamespace(footprint=FOOTPRINTS["hexagon"], poses=inputs.path_poses(rng, N, -half / 2, half / 2),
                             edges=maps[i % 2][0], obst_off=maps[i % 2][1]) for i in range(k)]
    a, b = api.Batch(insts, mbar=mbar), api.Batch(insts, mbar=mbar, exhaustive=True)
    assert all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(a.run(), b.run()))
    ms = [_time(torch, x.run, 5) for x in (a, b)]
    a.close()
    b.close()
    print(mbar, k, N, M, "default, full:", [round(1e3 * t, 1) for t in ms], flush=True)
    assert ms[0] <= 1.25 * ms[1], ms


@pytest.mark.parametrize("m", [3, 6])
@pytest.mark.parametrize("mbar,N,M", [(8, 1000, 1100), (8, 200, 16384), (8, 16, 250000), (8, 5, 1000000),
                                      (16, 50, 60000), (16, 9, 250000), (4, 50, 60000)])
def test_plain_call_on_wide_obstacles(m, mbar, N, M):
    rng = np.random.default_rng(10)
    t = np.arange(m) * 2 * np.pi / m
    fp = (0.5 * np.stack([np.cos(t), np.sin(t)], 1)).astype(np.float32)
    _plain(fp, N, M, *_octagons(rng, M, mbar, HALF * np.sqrt(M / 16384)), mbar)
