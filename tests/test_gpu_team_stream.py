"""GPU parity of the one-dimensional streams whose teams own ranges of
consecutive iterations (static, static chunk, dynamic, guided): AXPY bit for
bit against the oracle (an iteration run twice, or not at all, changes y),
SUM of every data type against exact host values, loops that start off a
16-byte boundary, ranges shorter than a vector, more teams than ranges, an
empty loop, and repeated launches (the claim counter re-arms itself).

Tolerance: AXPY, integers, maxima and minima exact; a float64 sum of n
values in another order is within n 2^-53 of the sum of their magnitudes.
"""
import numpy as np
import pytest

import synth
from oracle import bodies
from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

OPS = {"sum": U.UPIR_RED_SUM, "max": U.UPIR_RED_MAX, "min": U.UPIR_RED_MIN}
SCHEDS = [(U.UPIR_SCHED_STATIC, 0), (U.UPIR_SCHED_STATIC_CHUNK, 3), (U.UPIR_SCHED_STATIC_CHUNK, 64),
          (U.UPIR_SCHED_DYNAMIC, 1), (U.UPIR_SCHED_DYNAMIC, 50), (U.UPIR_SCHED_GUIDED, 1), (U.UPIR_SCHED_GUIDED, 9)]


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


@pytest.mark.parametrize("pol,chunk", SCHEDS + [(U.UPIR_SCHED_AUTO, 0)])
@pytest.mark.parametrize("n,off,T,Uu", [(0, 0, 3, 64), (1, 3, 0, 0), (3, 1, 2, 64), (4099, 1, 7, 96), (100003, 2, 0, 0),
                                        (100003, 0, 33, 1024), (300001, 3, 300, 64)])
def test_axpy(ctx, pol, chunk, n, off, T, Uu):
    print(f"axpy pol={pol} chunk={chunk} n={n} off={off} T={T} U={Uu}", flush=True)
    x, y = synth.uniform_pm1(51, 0, n + off + 2), synth.uniform_pm1(51, 1, n + off + 2)
    sched = H.make_sched(pol, chunk) if pol != U.UPIR_SCHED_AUTO else None
    for op in (None, "max", "min"):
        tx, ty = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        red = H.make_red(OPS[op], r.data_ptr(), init={"max": -9.0, "min": 9.0}[op]) if op else None
        lp = ctx.loop(U.UPIR_BODY_AXPY, U.upir_axpy_args(2.5, 0, tx.data_ptr(), ty.data_ptr()), [(off, off + n, 1)],
                      sched, red)
        want = y.copy()
        for _ in range(3):
            ctx.launch(lp, H.make_spmd(T, Uu))
            want[off:off + n] = bodies.axpy(2.5, x[off:off + n], want[off:off + n])
        ctx.sync()
        ctx.free(lp)
        assert np.array_equal(ty.cpu().numpy(), want)
        if op == "max":
            assert r.item() == max([-9.0] + [float(v) for v in want[off:off + n]])
        if op == "min":
            assert r.item() == min([9.0] + [float(v) for v in want[off:off + n]])


@pytest.mark.parametrize("dtype", ["f32", "f64", "i32", "i64"])
@pytest.mark.parametrize("pol,chunk", SCHEDS + [(U.UPIR_SCHED_AUTO, 0)])
@pytest.mark.parametrize("n,off,T,Uu", [(0, 0, 2, 64), (5, 1, 0, 0), (70001, 1, 5, 100), (300001, 0, 0, 0)])
def test_sum(ctx, dtype, pol, chunk, n, off, T, Uu):
    print(f"sum {dtype} pol={pol} chunk={chunk} n={n} off={off} T={T} U={Uu}", flush=True)
    if dtype[0] == "f":
        v = synth.uniform_pm1(52, 0, n + off).astype(np.float32 if dtype == "f32" else np.float64)
    else:
        v = synth.int_range(52, 0, n + off, -10 ** 9, 10 ** 9).astype(np.int32 if dtype == "i32" else np.int64)
    t = torch.from_numpy(v).cuda() if n + off else torch.zeros(1, device="cuda")
    sched = H.make_sched(pol, chunk) if pol != U.UPIR_SCHED_AUTO else None
    dt = {"f32": U.UPIR_DT_F32, "f64": U.UPIR_DT_F64, "i32": U.UPIR_DT_I32, "i64": U.UPIR_DT_I64}[dtype]
    part = v[off:]
    for op in ("sum", "max", "min"):
        if op == "sum" and dtype == "f32":
            continue
        r = torch.zeros(1, dtype=torch.float64 if dtype[0] == "f" else torch.int64, device="cuda")
        lp = ctx.loop(U.UPIR_BODY_SUM, U.upir_sum_args(t.data_ptr(), dt, 0), [(off, off + n, 1)], sched,
                      H.make_red(OPS[op], r.data_ptr(), init=1.0))
        for _ in range(3):
            ctx.launch(lp, H.make_spmd(T, Uu))
        ctx.sync()
        ctx.free(lp)
        got = r.item()
        if op == "sum":
            want = 1 + (sum(int(e) for e in part) if dtype[0] == "i" else bodies.sum_f64(part))
            bound = 0 if dtype[0] == "i" else (n + 1) * 2.0 ** -53 * (1 + bodies.sum_abs_f64(part))
            assert abs(got - want) <= bound
        else:
            assert got == (max if op == "max" else min)([1] + [e.item() for e in part])


@pytest.mark.parametrize("T", [1, 63, 64, 95, 96, 255, 256, 257])
@pytest.mark.parametrize("pol", [U.UPIR_SCHED_DYNAMIC, U.UPIR_SCHED_GUIDED])
def test_claim_queues(ctx, pol, T):
    # one to eight claim counters, ranges fewer and more than teams; each
    # launch starts from the counters that the one before re-armed
    for n in (0, 64, 64 * T - 1, 64 * T + 1, 64 * 7 * T + 33):
        x, y = synth.uniform_pm1(52, 0, n + 1), synth.uniform_pm1(52, 1, n + 1)
        tx, ty = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
        lp = ctx.loop(U.UPIR_BODY_AXPY, U.upir_axpy_args(2.5, 0, tx.data_ptr(), ty.data_ptr()), [(0, n, 1)],
                      H.make_sched(pol, 1))
        sp = H.make_spmd(T, 64)
        want = y.copy()
        for _ in range(4):
            ctx.launch(lp, sp)
            want[:n] = bodies.axpy(2.5, x[:n], want[:n])
        ctx.sync()
        ctx.free(lp)
        assert np.array_equal(ty.cpu().numpy(), want), (n, T)


@pytest.mark.parametrize("n", [(8 << 20) - 1, (8 << 20) + 1])
def test_static_default_teams(ctx, n):
    # either side of the size from which static blocks are one pass long
    x, y = synth.uniform_pm1(53, 0, n), synth.uniform_pm1(53, 1, n)
    tx, ty = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    lp = ctx.loop(U.UPIR_BODY_AXPY, U.upir_axpy_args(2.5, 0, tx.data_ptr(), ty.data_ptr()), [(0, n, 1)],
                  H.make_sched(U.UPIR_SCHED_STATIC))
    ctx.launch(lp)
    ctx.sync()
    ctx.free(lp)
    assert np.array_equal(ty.cpu().numpy(), bodies.axpy(2.5, x, y))
