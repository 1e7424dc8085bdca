"""GPU parity of the one-dimensional streams on teams of one, two and three
units: at each end of a range up to three elements lie outside its 16-byte
accesses, more than such a team has units. Every policy, data type, offset
from a 16-byte boundary and remainder modulo a vector, against the oracle (an
iteration run twice, or not at all, changes y; the extreme values of the
reductions sit in the ends).

Tolerance: AXPY, integers, maxima and minima exact; a float64 sum of n values
in another order is within n 2^-53 of the sum of their magnitudes.
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
SCHEDS = [(U.UPIR_SCHED_STATIC, 0), (U.UPIR_SCHED_STATIC_CHUNK, 3), (U.UPIR_SCHED_STATIC_CHUNK, 7),
          (U.UPIR_SCHED_DYNAMIC, 1), (U.UPIR_SCHED_DYNAMIC, 5), (U.UPIR_SCHED_GUIDED, 1), (U.UPIR_SCHED_GUIDED, 3)]
SPMD = [(1, 1), (1, 2), (4, 1), (3, 2), (5, 3)]
NS = [1, 2, 3, 7, 1000, 1001, 1002, 1003]


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


def check_axpy(ctx, pol, chunk, T, Uu):
    print(f"axpy pol={pol} chunk={chunk} T={T} U={Uu}", flush=True)
    for n in NS:
        for off in range(4):
            x, y = synth.uniform_pm1(61, 0, n + off + 2), synth.uniform_pm1(61, 1, n + off + 2)
            for op in (None, "max", "min"):
                tx, ty = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
                r = torch.zeros(1, dtype=torch.float64, device="cuda")
                red = H.make_red(OPS[op], r.data_ptr(), init={"max": -9.0, "min": 9.0}[op]) if op else None
                lp = ctx.loop(U.UPIR_BODY_AXPY, U.upir_axpy_args(2.5, 0, tx.data_ptr(), ty.data_ptr()),
                              [(off, off + n, 1)], H.make_sched(pol, chunk), red)
                want = y.copy()
                for _ in range(2):
                    ctx.launch(lp, H.make_spmd(T, Uu))
                    want[off:off + n] = bodies.axpy(2.5, x[off:off + n], want[off:off + n])
                ctx.sync()
                ctx.free(lp)
                assert np.array_equal(ty.cpu().numpy(), want), (n, off, op)
                if op:
                    assert r.item() == float(getattr(want[off:off + n], op)()), (n, off, op)


def check_sum(ctx, dtype, pol, chunk, T, Uu):
    print(f"sum {dtype} pol={pol} chunk={chunk} T={T} U={Uu}", flush=True)
    dt = {"f32": U.UPIR_DT_F32, "f64": U.UPIR_DT_F64, "i32": U.UPIR_DT_I32, "i64": U.UPIR_DT_I64}[dtype]
    for n in NS:
        for off in range(4):
            if dtype[0] == "f":
                v = synth.uniform_pm1(62, 0, n + off).astype(np.float32 if dtype == "f32" else np.float64)
            else:
                v = synth.int_range(62, 0, n + off, -10 ** 9, 10 ** 9).astype(np.int32 if dtype == "i32" else np.int64)
            # the largest and the smallest value among the last and the first three elements
            v[off + n - 1 - min(n % 3, n - 1)] = 2 * 10 ** 9
            v[off + min(off % 3, n - 1)] = -2 * 10 ** 9
            t = torch.from_numpy(v).cuda()
            part = v[off:]
            for op in ("sum", "max", "min"):
                if op == "sum" and dtype == "f32":
                    continue  # keeps the schedule's order: another kernel
                r = torch.zeros(1, dtype=torch.float64 if dtype[0] == "f" else torch.int64, device="cuda")
                lp = ctx.loop(U.UPIR_BODY_SUM, U.upir_sum_args(t.data_ptr(), dt, 0), [(off, off + n, 1)],
                              H.make_sched(pol, chunk), H.make_red(OPS[op], r.data_ptr(), init=1.0))
                for _ in range(2):
                    ctx.launch(lp, H.make_spmd(T, Uu))
                ctx.sync()
                ctx.free(lp)
                got = r.item()
                if op == "sum":
                    want = 1 + (sum(int(e) for e in part) if dtype[0] == "i" else bodies.sum_f64(part))
                    bound = 0 if dtype[0] == "i" else (n + 1) * 2.0 ** -53 * (1 + bodies.sum_abs_f64(part))
                    assert abs(got - want) <= bound, (n, off, op)
                else:
                    assert got == (max if op == "max" else min)([1] + [e.item() for e in part]), (n, off, op)


@pytest.mark.parametrize("pol,chunk", SCHEDS)
@pytest.mark.parametrize("T,Uu", SPMD)
def test_axpy(ctx, pol, chunk, T, Uu):
    check_axpy(ctx, pol, chunk, T, Uu)


@pytest.mark.parametrize("dtype", ["f32", "f64", "i32", "i64"])
@pytest.mark.parametrize("pol,chunk", SCHEDS)
@pytest.mark.parametrize("T,Uu", SPMD)
def test_sum(ctx, dtype, pol, chunk, T, Uu):
    check_sum(ctx, dtype, pol, chunk, T, Uu)


# chunk 4 over the flat unit number: the launch as a whole has one to three units
@pytest.mark.parametrize("T,Uu", [(1, 1), (1, 2), (2, 1), (1, 3), (3, 1)])
def test_chunk4(ctx, T, Uu):
    check_axpy(ctx, U.UPIR_SCHED_STATIC_CHUNK, 4, T, Uu)
    check_sum(ctx, "f32", U.UPIR_SCHED_STATIC_CHUNK, 4, T, Uu)
