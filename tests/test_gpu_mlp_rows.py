"""Every row counts in the screener's gradient: with targets that all rows but one
meet, the gradient is that row's own."""
import numpy as np
import pytest

from oracle import mlp_oracle as mo
from paper_2607_04310_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,rows", [(1, (0,)), (65, (0, 63, 64)), (16385, (16383, 16384)),
                                    (33000, (0, 15, 16, 47, 63, 64, 191, 192, 16384, 24575, 32767, 32768,
                                             32999))])
def test_one_row_off(B, rows):
    """The row is one whose pre-activations stay away from zero.  The oracle rounds
    the same operands to BF16; a rounding that falls the other way is 2^-8 of an
    operand, and the other rows' residuals are FP32 rounding."""
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(B)
    th = inputs.mlp_init_params(B)
    X = rng.uniform(-1.5, 1.5, (B, 4)).astype(np.float32)
    tries = rng.uniform(-1.5, 1.5, (4000, 4)).astype(np.float32)
    _, c = mo.forward(th, tries)
    x = tries[np.argmax(np.minimum(np.abs(c["h1pre"]).min(1), np.abs(c["h2pre"]).min(1)))]
    thd = torch.tensor(th, device="cuda")
    for r in rows:
        Xr = X.copy()
        Xr[r] = x
        Xd = torch.tensor(Xr, device="cuda")
        T = api.mlp_forward(thd, Xd)
        T[r] -= 1.0
        g, loss = api.mlp_grad(thd, Xd, T)
        y, _ = mo.forward(th, x[None])
        want = mo.backward(th, x[None], y - 1.0) / B
        for name, a, b in zip(("W1", "b1", "W2", "b2", "w3", "b3"), mo.unpack(g.cpu().numpy()), mo.unpack(want)):
            a, b = np.asarray(a), np.asarray(b)
            assert np.abs(a - b).max() <= 2.0 ** -7 * np.abs(b).max(), (r, name)
        assert abs(float(loss) * B - 1.0) <= 1e-3, r
