"""GPU parity of the tiled Jacobi and 7 x 7 filter strips on grids whose
pitch is no multiple of four and whose first element is off a 16-byte
boundary: bit for bit against the oracle, for tiles ragged on all sides, one
or two columns, every tile height and one or several wavefronts per tile;
nothing outside the loop box is written.
"""
import numpy as np
import pytest

import synth
from oracle import bodies
from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(40, 257), (131, 1021), (9, 515), (300, 9), (67, 770)]
SCHEDS = [(None, 0), (4, 64), (8, 256), (16, 192), (32, 512), (64, 128)]


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


def placed(a, off):
    t = torch.full((a.size + 8,), -7.0, device="cuda")
    t[off:off + a.size] = torch.from_numpy(np.ascontiguousarray(a)).cuda().reshape(-1)
    return t, t.data_ptr() + 4 * off


@pytest.mark.parametrize("th,units", SCHEDS)
@pytest.mark.parametrize("shape", SHAPES)
def test_jacobi(ctx, shape, th, units):
    print(f"jacobi {shape} tile {th} units {units}", flush=True)
    rows, cols = shape
    u = synth.uniform_01(61, 0, rows * cols).reshape(shape)
    want = u * 0 - 7
    full = bodies.jacobi5_sweep_f32(u)
    want[1:-1, 1:-1] = full[1:-1, 1:-1]
    res = bodies.update_f64(full, u, "max")
    sched = H.make_sched(U.UPIR_SCHED_STATIC, tile=(th, 256)) if th else None
    for off in (0, 1, 3):
        for async_ in (False, True):
            src, ps = placed(u, off)
            dst, pd = placed(np.full(shape, -7.0, np.float32), (off + 2) % 4)
            r = torch.zeros(1, dtype=torch.float64, device="cuda")
            lp = ctx.loop(U.UPIR_BODY_JACOBI5, U.upir_jacobi5_args(ps, pd, cols), [(1, rows - 1, 1), (1, cols - 1, 1)],
                          sched, H.make_red(U.UPIR_RED_MAX, r.data_ptr(), async_=async_))
            ctx.launch(lp, H.make_spmd(0, units))
            ctx.sync()
            ctx.free(lp)
            out = dst.cpu().numpy()
            at = (off + 2) % 4
            assert np.array_equal(out[at:at + u.size].reshape(shape), want)
            assert (out[:at] == -7).all() and (out[at + u.size:] == -7).all()
            assert r.item() == res


@pytest.mark.parametrize("th,units", SCHEDS)
@pytest.mark.parametrize("shape", SHAPES)
def test_filter7(ctx, shape, th, units):
    print(f"filter7 {shape} tile {th} units {units}", flush=True)
    rows, cols = shape
    u = synth.uniform_pm1(62, 0, rows * cols).reshape(shape)
    w = synth.uniform_pm1(62, 1, 49).reshape(7, 7) * np.float32(0.25)
    want = bodies.filter7(u, w, np.full(shape, -7.0, np.float32))
    tw = torch.from_numpy(w).cuda()
    sched = H.make_sched(U.UPIR_SCHED_STATIC, tile=(th, 256)) if th else None
    for off in (0, 1, 3):
        src, ps = placed(u, off)
        dst, pd = placed(np.full(shape, -7.0, np.float32), (off + 2) % 4)
        lp = ctx.loop(U.UPIR_BODY_FILTER7, U.upir_filter7_args(ps, pd, tw.data_ptr(), cols),
                      [(3, rows - 3, 1), (3, cols - 3, 1)], sched)
        ctx.launch(lp, H.make_spmd(0, units))
        ctx.sync()
        ctx.free(lp)
        out = dst.cpu().numpy()
        at = (off + 2) % 4
        assert np.array_equal(out[at:at + u.size].reshape(shape), want)
        assert (out[:at] == -7).all() and (out[at + u.size:] == -7).all()
