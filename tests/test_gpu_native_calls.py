"""The native calls take every form of argument that the Python API takes, with
the same results and the same errors."""
import numpy as np
import pytest

from paper_2607_04310_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture()
def scene():
    import torch
    from paper_2607_04310_amd import api
    inst = inputs.c1(0)
    es = api.EdgeSet(inst.edges, inst.obst_off)
    return api, torch, inst, es, torch.tensor(inst.poses, device="cuda")


def _same(a, b):
    import torch
    torch.cuda.synchronize()
    return all(x.dtype == y.dtype and x.shape == y.shape and x.device == y.device
               and torch.equal(x, y) for x, y in zip(a, b))


def test_footprint_and_pose_forms(scene):
    api, torch, inst, es, poses = scene
    want = api.psdf_grad(inst.footprint, poses, es)
    fp = inst.footprint
    for form in (fp.tolist(), fp.astype(np.float64), torch.tensor(fp), fp.ravel(), np.asfortranarray(fp),
                 fp.astype(">f4"), np.repeat(fp, 2, axis=0)[::2]):
        assert _same(api.psdf_grad(form, poses, es), want)
    wide = torch.zeros(poses.shape[0], 5, device="cuda")
    wide[:, 1:4] = poses
    grad = poses.clone().requires_grad_(True)
    for p in (wide[:, 1:4], poses.t().contiguous().t(), grad):
        got = api.psdf_grad(fp, p, es)
        assert _same(got, want) and not got[0].requires_grad
    assert _same(api.psdf_grad(fp, poses[:0], es), [t[:0] for t in want])


def test_out_ws_host_and_streams(scene):
    api, torch, inst, es, poses = scene
    want = api.psdf_grad(inst.footprint, poses, es)
    out = tuple(torch.empty_like(t) for t in want)
    got = api.psdf_grad(inst.footprint, poses, es, api.Params(), list(out),
                        api.workspace(poses.shape[0], es.M, "cuda"))
    assert all(g is o for g, o in zip(got, out)) and _same(got, want)
    hj, _ = api.psdf_constraints(inst.footprint, poses, es, 0.01)
    host = torch.empty(poses.shape[0], 4, pin_memory=True)
    api.psdf_constraints(inst.footprint, poses, es, 0.01, host=host)
    torch.cuda.synchronize()
    assert torch.equal(host, hj.cpu())
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        late = torch.empty_like(poses)
        late.copy_(poses)          # ordered before the call on this stream only
        got = api.psdf_grad(inst.footprint, late, es)
    s.synchronize()
    assert _same(got, want)
    assert _same(api.psdf_eval(inst.footprint, poses, es), want[:3] + want[4:])


def test_errors(scene):
    api, torch, inst, es, poses = scene
    fp = inst.footprint
    for bad in (poses.cpu(), poses.double(), poses[:, :2], poses[0], inst.poses):
        with pytest.raises(AssertionError):
            api.psdf_grad(fp, bad, es)
    with pytest.raises(AttributeError):
        api.psdf_grad(fp, inst.poses.tolist(), es)
    with pytest.raises(ValueError):
        api.psdf_grad(np.zeros(7, np.float32), poses, es)
    with pytest.raises(api.PsdfError) as e:
        api.psdf_grad(fp[[0, 2, 1, 3]], poses, es)
    assert e.value.code == -2 and "convex" in str(e.value)
    with pytest.raises(api.PsdfError) as e:
        api.psdf_grad(np.zeros((0, 2), np.float32), poses, es)
    assert e.value.code == -2
    with pytest.raises(ValueError):
        api.psdf_grad(fp, poses, es, out=(poses, poses))
    for host in (torch.empty(3, 4), torch.empty(poses.shape[0], 4, dtype=torch.float64),
                 torch.empty(4, poses.shape[0]).t(), torch.empty(poses.shape[0], 4, device="cuda")):
        with pytest.raises(ValueError):
            api.psdf_constraints(fp, poses, es, 0.01, host=host)
    with pytest.raises(api.PsdfError):
        api.psdf_constraints(fp, poses, es, float("nan"))
    with pytest.raises(api.PsdfError) as e:
        api.psdf_grad(fp, poses, es, ws=torch.empty(8, dtype=torch.uint8, device="cuda"))
    assert e.value.code == -5
    es.stage()
    with pytest.raises(api.PsdfError) as e:
        api.psdf_grad(fp, poses, es, api.Params(eps=1e-3))
    assert e.value.code == -1
    es.ax = es.ax.clone()
    with pytest.raises(api.PsdfError):
        api.psdf_grad(fp, poses, es)


def test_encode_mask_forms(scene):
    api, torch, inst, es, poses = scene
    rng = np.random.default_rng(2)
    A, B = (torch.tensor(rng.normal(size=(37, 6, 2)).astype(np.float32), device="cuda")
            for _ in range(2))
    S = torch.tensor(rng.random((37, 6)) < 0.6, device="cuda")
    want = api.psdf_encode_padded(A, B, S)
    keep = S.cpu().numpy()
    np.testing.assert_array_equal(want.ax.cpu().numpy(), A.cpu().numpy()[keep][:, 0])
    np.testing.assert_array_equal(want.obst_off.cpu().numpy(), inputs.csr_offsets(keep.sum(1)))
    for a, b, s in ((A.double(), B.double(), S.to(torch.uint8)), (A, B, S.long()),
                    (A.transpose(0, 1).contiguous().transpose(0, 1), B, S.t().contiguous().t())):
        got = api.psdf_encode_padded(a, b, s)
        assert got.E == want.E and got.M == want.M and got.mbar == want.mbar
        assert _same([got.ax, got.ay, got.bx, got.by, got.obst_off],
                     [want.ax, want.ay, want.bx, want.by, want.obst_off])
