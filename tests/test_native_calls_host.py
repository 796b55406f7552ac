"""The native calls on a host without a usable GPU: every one raises what torch
raises, and none ends the interpreter (each runs in a process of its own)."""
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="host tensors are refused by "
                                "the missing device here; with one they would reach the kernels")

CALLS = {
    "mlp_train_step": """th = torch.zeros(4545)
api.mlp_train_step(th, th.clone(), th.clone(), 1, 1e-3, torch.zeros(4, 4), torch.zeros(4))""",
    "encode_padded": """A = torch.zeros(2, 3, 2)
api.psdf_encode_padded(A, A, torch.ones(2, 3, dtype=torch.bool))""",
    "stage": """api.EdgeSet(np.zeros((4, 4), np.float32), [0, 4], device="cpu").stage()""",
}


def _run(body):
    code = f"""import numpy as np, torch
from paper_2607_04310_amd import api
try:
    {body.replace(chr(10), chr(10) + "    ")}
except Exception as e:
    print(type(e).__name__, e)
else:
    print("no exception")
"""
    return subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)


@pytest.mark.parametrize("name", sorted(CALLS))
def test_no_device(name):
    r = _run(CALLS[name])
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    assert r.stdout.startswith("RuntimeError") and "GPU" in r.stdout, r.stdout


@pytest.mark.parametrize("step", ["500.0", "np.float32(7)", "torch.tensor(3.0)", "True", "'12'"])
def test_step_and_rate_convert_as_int_and_float(step):
    """step and lr are int(step) and float(lr): any of these forms gets as far
    as the missing device."""
    r = _run(f"""th = torch.zeros(4545)
api.mlp_train_step(th, th.clone(), th.clone(), {step}, '1e-3', torch.zeros(4, 4), torch.zeros(4))""")
    assert r.returncode == 0 and r.stdout.startswith("RuntimeError"), (r.stdout, r.stderr[-300:])


def test_exception_types():
    """What torch raises keeps its class (a 0-dimensional X has no rows)."""
    r = _run("""th = torch.zeros(4545)
api.mlp_train_step(th, th.clone(), th.clone(), 1, 1e-3, torch.tensor(1.0), torch.zeros(1))""")
    assert r.returncode == 0 and r.stdout.startswith("IndexError"), (r.stdout, r.stderr[-300:])
