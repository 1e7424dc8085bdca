"""Tasks of one and of many tiles in the batched executor.

A finished task's tiles are folded by one wavefront, 64 tiles to a group and
four groups to a pass, a task of one tile without going through memory; its
successors are released one per lane; AXPY without a reduction starts its
16-byte accesses at any element. Tile counts around each of those edges,
every operator, every element offset. The data are small whole numbers, so
every result is exact and compared with ==.
"""
import numpy as np
import pytest

from oracle import tasks as otasks
from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TILE = 256
NP_OP = {U.UPIR_RED_SUM: np.sum, U.UPIR_RED_MAX: np.max, U.UPIR_RED_MIN: np.min}


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available()
    U.lib()
    s = torch.cuda.Stream()
    prev = torch.cuda.current_stream()
    torch.cuda.set_stream(s)
    c = H.Context(0, stream=s)
    yield c
    c.close()
    torch.cuda.set_stream(prev)


@pytest.mark.parametrize("fan", [0, 3, 70])
@pytest.mark.parametrize("op", [None, U.UPIR_RED_SUM, U.UPIR_RED_MAX, U.UPIR_RED_MIN])
@pytest.mark.parametrize("n", [1, TILE, TILE + 1, 64 * TILE, 64 * TILE + 1, 256 * TILE, 256 * TILE + 5, 300 * TILE])
def test_task_tiles(ctx, n, op, fan):
    # task 0: y += 2 x, reduced with op; tasks 1 .. fan: sums of y after it
    rng = np.random.RandomState(n % 1000 + fan)
    off = (n + fan) % 4
    x = rng.randint(-9, 10, n + 4).astype(np.float32)
    y = rng.randint(-9, 10, n + 4).astype(np.float32)
    tx, ty = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    res = torch.zeros(1 + fan, dtype=torch.float64, device="cuda")
    tok = torch.zeros(1 + fan, dtype=torch.int64, device="cuda")
    sched = H.make_sched(U.UPIR_SCHED_AUTO, tile=(TILE,))
    xp, yp, rp = tx.data_ptr() + 4 * off, ty.data_ptr() + 4 * off, res.data_ptr()
    loops = [ctx.loop(U.UPIR_BODY_AXPY, U.upir_axpy_args(2.0, 0, xp, yp), [(0, n, 1)], sched,
                      H.make_red(op, rp) if op is not None else None)]
    for j in range(fan):
        loops.append(ctx.loop(U.UPIR_BODY_SUM, U.upir_sum_args(yp, U.UPIR_DT_F32, 0), [(0, n, 1)], sched,
                              H.make_red(U.UPIR_RED_SUM, rp + 8 * (1 + j))))
    for j, lp in enumerate(loops):
        ctx.task(lp, [(yp, U.UPIR_DEP_INOUT if j == 0 else U.UPIR_DEP_IN)])
    ctx.set_trace(tok.data_ptr(), 0, 0)
    g = ctx.taskwait_graph(U.UPIR_TASKWAIT_BATCHED)
    ctx.set_trace()
    want_y = y.copy()
    for _ in range(3):  # replays of one graph: y goes on growing
        ctx.graph_launch(g)
        ctx.sync()
        want_y[off:off + n] += 2 * x[off:off + n]
        assert np.array_equal(ty.cpu().numpy(), want_y)
        got = res.cpu().numpy()
        part = want_y[off:off + n].astype(np.float64)
        if op is not None:
            assert got[0] == NP_OP[op](np.append(part, 0.0))  # the initial value takes part
        assert np.all(got[1:] == part.sum())
        preds = [[]] + [[0]] * fan
        assert [int(v) & (2 ** 64 - 1) for v in tok.cpu().numpy()] == otasks.tokens(preds)
    ctx.graph_destroy(g)
    for lp in loops:
        ctx.free(lp)
