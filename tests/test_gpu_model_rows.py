"""GPU parity of the cost model's row kernel at the row counts where it can go
wrong: fewer rows than one iteration takes, remainders, one row per wavefront
and many, more wavefronts than the update kernel's runs. Predictions, the
loss and every gradient against the float64 oracle; one Adam step.

Tolerance: float32 sums of at most 65 terms in the forward pass and of n
terms in the gradients, in some order: normwise 1e-5, as for the other tests
of this network.
"""
import ctypes as C

import numpy as np
import pytest

import synth
from oracle import mlp
from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    U.lib()
    s = torch.cuda.Stream()
    prev = torch.cuda.current_stream()
    torch.cuda.set_stream(s)  # torch's work and the library's are ordered on one stream
    c = H.Context(0, stream=s)
    yield c
    c.close()
    torch.cuda.set_stream(prev)


SHAPES = {"W1": (64, 32), "b1": (64,), "W2": (64, 64), "b2": (64,), "W3": (1, 64), "b3": (1,)}


def rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b)


def unflat(v):
    P, o = {}, 0
    for k in mlp.NAMES:
        n = int(np.prod(SHAPES[k]))
        P[k] = np.asarray(v[o:o + n], np.float64).reshape(SHAPES[k])
        o += n
    return P


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 255, 257, 1023, 1030, 4097, 5001])
def test_rows(ctx, n):
    print(f"model rows {n}", flush=True)
    p = np.empty(U.UPIR_MLP_PARAMS, np.float32)
    U.upir_model_init(ctx.h, 77)
    U.upir_model_get_params(ctx.h, p.ctypes.data_as(C.POINTER(C.c_float)))
    p += synth.uniform_pm1(70, 0, p.size) * np.float32(0.05)  # biases that are not zero
    U.upir_model_set_params(ctx.h, p.ctypes.data_as(C.POINTER(C.c_float)))
    x = synth.uniform_01(70, 1, n * 32).reshape(n, 32)
    t = synth.uniform_01(70, 2, n) * np.float32(8)
    tx, tt = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    y = torch.full((n + 4,), -7.0, device="cuda")
    U.upir_model_forward(ctx.h, tx.data_ptr(), n, y.data_ptr())
    grad = torch.zeros(U.UPIR_MLP_PARAMS, device="cuda")
    loss = C.c_float()
    U.upir_model_step(ctx.h, tx.data_ptr(), tt.data_ptr(), n, 1e-3, 1, grad.data_ptr(), C.byref(loss))
    got = y.cpu().numpy()
    assert (got[n:] == -7.0).all()
    P = unflat(p)
    want, _ = mlp.forward(P, x)
    assert rel(got[:n], want) <= 1e-5
    assert abs(loss.value - mlp.loss(P, x, t)) <= 1e-5 * mlp.loss(P, x, t)
    want_grad, got_grad = mlp.backward(P, x, t), unflat(grad.cpu().numpy())
    for k in mlp.NAMES:
        assert rel(got_grad[k], want_grad[k]) <= 1e-5, k
    after = np.empty_like(p)
    U.upir_model_get_params(ctx.h, after.ctypes.data_as(C.POINTER(C.c_float)))
    g = grad.cpu().numpy().astype(np.float64)  # the first step moves every parameter by lr g / (|g| + eps)
    assert np.abs(after - (p - 1e-3 * g / (np.abs(g) + 1e-8))).max() <= 1e-6
