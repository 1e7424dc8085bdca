"""GPU parity of the cost model's forward pass at the row counts around the
one from which it takes a row per thread: predictions against the float64
oracle, nothing written past them.

Tolerance: float32 sums of at most 65 terms: normwise 1e-5, as for the other
tests of this network.
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
SHAPES = {"W1": (64, 32), "b1": (64,), "W2": (64, 64), "b2": (64,), "W3": (1, 64), "b3": (1,)}


@pytest.mark.parametrize("n", [(96 << 10) - 1, 96 << 10, (96 << 10) + 1, 120001])
def test_forward_of_many_rows(n):
    print(f"model forward {n}", flush=True)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), H.Context(0, stream=s) as ctx:
        p = np.empty(U.UPIR_MLP_PARAMS, np.float32)
        U.upir_model_init(ctx.h, 78)
        U.upir_model_get_params(ctx.h, p.ctypes.data_as(C.POINTER(C.c_float)))
        p += synth.uniform_pm1(71, 0, p.size) * np.float32(0.05)  # biases that are not zero
        U.upir_model_set_params(ctx.h, p.ctypes.data_as(C.POINTER(C.c_float)))
        x = synth.uniform_01(71, 1, n * 32).reshape(n, 32)
        tx, y = torch.from_numpy(x).cuda(), torch.full((n + 300,), -7.0, device="cuda")
        U.upir_model_forward(ctx.h, tx.data_ptr(), n, y.data_ptr())
        ctx.sync()
        got = y.cpu().numpy()
    P, o = {}, 0
    for k in mlp.NAMES:
        m = int(np.prod(SHAPES[k]))
        P[k] = p[o:o + m].astype(np.float64).reshape(SHAPES[k])
        o += m
    want, _ = mlp.forward(P, x)
    assert (got[n:] == -7.0).all()
    assert np.linalg.norm(got[:n] - want) <= 1e-5 * np.linalg.norm(want)
