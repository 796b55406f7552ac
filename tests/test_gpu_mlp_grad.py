"""The screener's gradient at the edges of its 64-row work-group iterations
(one row, a row more or less than an iteration, than the 256 work-groups, a
ragged last round), and on parameters and rows that start at any float
address."""
import numpy as np
import pytest

from oracle import mlp_oracle as mo
from paper_2607_04310_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 63, 64, 65, 16384, 16385, 33000])
@pytest.mark.parametrize("shift", [0, 1])
def test_grad_at_the_edges(B, shift):
    """BF16 rounds each operand by at most 2^-9 of itself and the oracle rounds
    the same operands: what is left are the products whose rounding falls the
    other way and the order of FP32 sums, well within 3 % of each block's
    largest entry."""
    import torch
    from paper_2607_04310_amd import api
    rng = np.random.default_rng(B)
    th = inputs.mlp_init_params(B)
    X = rng.uniform(-1.5, 1.5, (B, 4)).astype(np.float32)
    T = rng.uniform(0, 2, B).astype(np.float32)

    def device(a):
        flat = torch.zeros(a.size + 4, device="cuda")
        flat[shift:shift + a.size] = torch.tensor(a.ravel(), device="cuda")
        return flat[shift:shift + a.size].view(a.shape)

    g, loss = api.mlp_grad(device(th), device(X), device(T))
    ref = mo.backward(th, X, T, bf16_on=True)
    for name, a, b in zip(("W1", "b1", "W2", "b2", "w3", "b3"), mo.unpack(g.cpu().numpy()),
                          mo.unpack(ref)):
        a, b = np.asarray(a), np.asarray(b)
        assert np.abs(a - b).max() <= 3e-2 * max(1e-6, np.abs(b).max()), name
    want = mo.loss(th, X, T, True)
    assert abs(float(loss) - want) <= 2e-2 * max(1e-6, want)
