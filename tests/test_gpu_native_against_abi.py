"""The native calls pass their arguments to the C ABI as they are: the adjoints, the
distance matrix with the caller's output and the training step give the bits that
the library gives when it is called directly, staged and not, with parameters of
their own."""
import ctypes

import numpy as np
import pytest

from paper_2607_04310_amd import inputs

pytestmark = pytest.mark.gpu


def _raw(name, *args):
    from paper_2607_04310_amd import _lib
    _lib.check(getattr(_lib.lib(), name)(*args))


@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("params", [None, dict(eta=50.0, eps_sat=1e-4)])
def test_adjoints_and_matrix(staged, params):
    import torch
    from paper_2607_04310_amd import _lib, api
    rng = np.random.default_rng(3)
    inst = inputs.c1(0)
    pr = None if params is None else api.Params(**params)
    es = api.EdgeSet(inst.edges, inst.obst_off)
    if staged:
        es.stage(pr)
    poses = torch.tensor(inst.poses, device="cuda")
    N = poses.shape[0]
    keys = api.psdf_grad(inst.footprint, poses, es, pr)[4]
    wide = torch.tensor(rng.normal(size=(N, 2)).astype(np.float32), device="cuda")
    fp, fpp, m = api._fp(inst.footprint)
    ec, pc = es.c(), (pr or api.Params()).c()
    for gout in (wide[:, 0], wide[:, 1].contiguous(), wide[:, 0].double()):
        g = gout.contiguous().to(torch.float32)
        want = torch.empty(N, 3, device="cuda")
        _raw("psdf_bwd", fpp, m, poses.data_ptr(), N, ctypes.byref(ec), ctypes.byref(pc), keys.data_ptr(),
             g.data_ptr(), want.data_ptr(), _lib.stream_handle())
        assert torch.equal(api.psdf_bwd(inst.footprint, poses, es, keys, gout, pr), want)
        # one stage at a time: the geometry adjoint's sums over stages are atomic
        for s in range(0, N, 7):
            one = torch.zeros(N, device="cuda")
            one[s] = g[s]
            ge, gf = torch.empty(es.E, 4, device="cuda"), torch.empty(m, 2, device="cuda")
            _raw("psdf_bwd_geometry", fpp, m, poses.data_ptr(), N, ctypes.byref(ec), ctypes.byref(pc),
                 keys.data_ptr(), one.data_ptr(), ge.data_ptr(), gf.data_ptr(), _lib.stream_handle())
            got = api.psdf_bwd_geometry(inst.footprint, poses, es, keys, one, pr)
            assert torch.equal(got[0], ge) and torch.equal(got[1], gf)
    want = torch.empty(N, es.M, device="cuda")
    _raw("psdf_sd_matrix", fpp, m, poses.data_ptr(), N, ctypes.byref(ec), ctypes.byref(pc), want.data_ptr(),
         _lib.stream_handle())
    out = torch.zeros(N, es.M, device="cuda")
    assert api.psdf_sd_matrix(inst.footprint, poses, es, pr, out=out) is out
    assert torch.equal(out, want) and torch.equal(api.psdf_sd_matrix(inst.footprint, poses, es, pr), want)


@pytest.mark.parametrize("B", [1, 65, 4096])
def test_training_step(B):
    import torch
    from paper_2607_04310_amd import _lib, api
    rng = np.random.default_rng(B)
    X = torch.tensor(rng.normal(size=(B, 4)).astype(np.float32), device="cuda")
    T = X[:, 0].contiguous()
    th = [torch.tensor(inputs.mlp_init_params(B), device="cuda") for _ in range(2)]
    m, v = ([torch.zeros_like(th[0]) for _ in range(2)] for _ in range(2))
    loss = [torch.zeros(1, device="cuda") for _ in range(2)]
    ws = torch.empty(int(_lib.lib().psdf_mlp_ws_bytes(B)), dtype=torch.uint8, device="cuda")
    for step in (1, 2, 700):
        _raw("psdf_mlp_train_step", th[0].data_ptr(), m[0].data_ptr(), v[0].data_ptr(), step, 1e-3,
             X.data_ptr(), T.data_ptr(), B, loss[0].data_ptr(), ws.data_ptr(), ws.numel(), _lib.stream_handle())
        api.mlp_train_step(th[1], m[1], v[1], step, 1e-3, X, T, loss=loss[1], ws=ws if step == 2 else None)
        for a, b in (th, m, v, loss):
            assert torch.equal(a, b), step
