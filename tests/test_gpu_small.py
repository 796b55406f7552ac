"""The one-launch form of small calls (up to 256 obstacles of at most four
edges), a quad of lanes per obstacle or a lane, around the sizes where it
changes, against the two-kernel form of the same set with empty obstacles
appended (an empty obstacle contributes nothing and moves no index): equal bit
for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _obstacles(rng, M, odd):
    """Closed polygons, segments and open pairs of edges; odd: also empty obstacles."""
    edges, off = [], [0]
    for i in range(M):
        c = rng.uniform(-3, 3, 2)
        kind = rng.integers(0, 5 if odd else 4)
        k = int(rng.integers(3, 5))
        ang = np.sort(rng.uniform(0, 2 * np.pi, k))
        P = c + rng.uniform(0.1, 0.6) * np.stack([np.cos(ang), np.sin(ang)], 1)
        if kind == 0:
            e = np.concatenate([P, np.roll(P, -1, 0)], 1)[:1]
        elif kind == 1:
            e = np.concatenate([P, np.roll(P, -1, 0)], 1)[:2]
        elif kind == 4:
            e = np.zeros((0, 4))
        else:
            e = np.concatenate([P, np.roll(P, -1, 0)], 1)
        edges.append(e.astype(np.float32))
        off.append(off[-1] + len(e))
    return np.concatenate(edges).astype(np.float32).reshape(-1, 4), np.array(off, np.int32)


@pytest.mark.parametrize("M,N", [(1, 1), (1, 9), (15, 40), (16, 3000), (17, 2048), (17, 2049),
                                 (64, 512), (64, 513), (65, 20), (127, 128), (128, 128),
                                 (128, 129), (129, 5)])
@pytest.mark.parametrize("m,hard", [(3, False), (6, True), (6, False), (11, False)])
def test_small_forms(M, N, m, hard):
    import paper_2607_04310_amd.api as api
    rng = np.random.default_rng([M, N, m])
    ang = 2 * np.pi * np.arange(m) / m
    fpv = np.stack([0.5 * np.cos(ang), 0.3 * np.sin(ang)], 1).astype(np.float32)
    par = api.Params(eta=float("inf") if hard else 50.0)
    poses = np.concatenate([rng.uniform(-3, 3, (N, 2)), rng.uniform(-4, 4, (N, 1))], 1)
    poses = poses.astype(np.float32)
    poses[N // 2, rng.integers(0, 3)] = np.nan if N > 1 else 0.0
    pt = torch.tensor(poses).cuda()
    for odd in (0, 1, 2):
        ed, off = _obstacles(rng, M, odd > 0)
        if len(ed) == 0:
            ed, off = _obstacles(rng, M, False)
        if odd == 2:   # a non-finite coordinate makes every stage NaN
            ed[len(ed) // 2, 1] = np.inf
        wide = np.concatenate([off, np.full(300, off[-1], np.int32)])
        a = api.psdf_grad(fpv, pt, api.EdgeSet(ed, off, 4), par)
        b = api.psdf_grad(fpv, pt, api.EdgeSet(ed, wide, 4), par)
        for x, y in zip(a[:4], b[:4]):
            assert x.cpu().numpy().tobytes() == y.cpu().numpy().tobytes()
        a = api.psdf_eval(fpv, pt, api.EdgeSet(ed, off, 4), par)
        for x, y in zip(a[:3], b[:3]):
            assert x.cpu().numpy().tobytes() == y.cpu().numpy().tobytes()
