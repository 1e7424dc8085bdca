"""GPU parity of the matvec kernels where they can go wrong: one, some and all
of a wavefront's rows together and the remainder, columns below, at and beyond
a block of 256 and a load group, pitches and starts off a 16-byte boundary, strided loops, a reduction.

Tolerance: float32 chains of `cols` products in some order, normwise 1e-5
as for the other matvec tests. A row's value does not depend on how many rows
run together, so the default and a one-row-at-a-time schedule agree bit for
bit where both run a wavefront per row.
"""
import numpy as np
import pytest

import synth
from oracle import bodies
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


def run(ctx, A, x, pad, off, dims, sched=None, spmd=None, red=None):
    rows, cols = A.shape
    buf = torch.full((off + rows * (cols + pad) + 4,), float("nan"), device="cuda")
    buf[off:off + rows * (cols + pad)].view(rows, cols + pad)[:, :cols] = torch.from_numpy(A).cuda()
    tx = torch.full((cols + off + 4,), float("nan"), device="cuda")
    tx[off:off + cols] = torch.from_numpy(x).cuda()
    y = torch.full((rows + 2,), -7.0, device="cuda")
    lp = ctx.loop(U.UPIR_BODY_MATVEC, U.upir_matvec_args(buf.data_ptr() + 4 * off, tx.data_ptr() + 4 * off, y.data_ptr(),
                                                         cols, cols + pad), dims, sched, red)
    ctx.launch(lp, spmd)
    ctx.sync()
    ctx.free(lp)
    out = y.cpu().numpy()
    assert (out[rows:] == -7.0).all()
    return out[:rows]


@pytest.mark.parametrize("rows,cols", [(1, 1), (3, 255), (70, 257), (33, 1025), (257, 3001), (90, 4099), (5, 20000)])
@pytest.mark.parametrize("T,Uu,static", [(0, 0, False), (2, 64, False), (3, 128, False), (300, 256, True), (9, 192, True)])  # static: contiguous rows
def test_rows(ctx, rows, cols, T, Uu, static):
    print(f"matvec {rows}x{cols} T={T} U={Uu} static={static}", flush=True)
    A = synth.uniform_pm1(71, 0, rows * cols).reshape(rows, cols)
    x = synth.uniform_pm1(71, 1, cols)
    want = bodies.matvec(A, x)
    sched = None if not T else (H.make_sched(U.UPIR_SCHED_STATIC) if static else H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 1))
    one = H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 2)  # its rows are not a fixed stride apart: one at a time
    for pad, off in ((0, 0), (3, 1), (5, 2)):
        got = run(ctx, A, x, pad, off, [(0, rows, 1)], sched, H.make_spmd(T, Uu))
        assert bodies.frob_rel(got, want) <= 1e-5
        if T and not static:
            assert np.array_equal(got, run(ctx, A, x, pad, off, [(0, rows, 1)], one, H.make_spmd(T, Uu)))


def test_strided_rows_and_reduction(ctx):
    rows, cols = 301, 700
    A = synth.uniform_pm1(72, 0, rows * cols).reshape(rows, cols)
    x = synth.uniform_pm1(72, 1, cols)
    full = bodies.matvec(A, x)
    for dims in ([(2, 300, 3)], [(300, 0, -7)]):
        idx = np.arange(*dims[0])
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        red = H.make_red(U.UPIR_RED_MAX, r.data_ptr(), init=-100.0)
        got = run(ctx, A, x, 1, 3, dims, H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 1), H.make_spmd(3, 128), red)
        assert bodies.frob_rel(got[idx], full[idx]) <= 1e-5
        rest = np.setdiff1d(np.arange(rows), idx)
        assert (got[rest] == -7.0).all()
        assert r.item() == float(got[idx].max())


@pytest.mark.parametrize("rows", [8, 9, 15, 16, 17, 24, 25, 28, 31, 32, 33, 40, 41, 47, 48, 63, 65])
def test_rows_left_over(ctx, rows):
    # eight wavefronts: some with four, three, two, one or no rows of a round
    cols = 1030
    A = synth.uniform_pm1(73, 0, rows * cols).reshape(rows, cols)
    x = synth.uniform_pm1(73, 1, cols)
    chunk1, one = H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 1), H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 2)
    got = run(ctx, A, x, 2, 1, [(0, rows, 1)], chunk1, H.make_spmd(8, 64))
    assert bodies.frob_rel(got, bodies.matvec(A, x)) <= 1e-5
    assert np.array_equal(got, run(ctx, A, x, 2, 1, [(0, rows, 1)], one, H.make_spmd(8, 64)))


@pytest.mark.parametrize("rows,cols", [(2100, 24000), (4096, 32770), (4694, 28600)])
def test_default_teams_of_large_matrices(ctx, rows, cols):
    # few rows, rows that come out even over the CUs, rows that do not
    A = torch.randn(rows, cols, device="cuda")
    x, y, z = torch.randn(cols, device="cuda"), torch.zeros(rows, device="cuda"), torch.zeros(rows, device="cuda")
    for out, sched, spmd in ((y, None, None), (z, H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 2), H.make_spmd(64, 256))):
        lp = ctx.loop(U.UPIR_BODY_MATVEC, U.upir_matvec_args(A.data_ptr(), x.data_ptr(), out.data_ptr(), cols, cols),
                      [(0, rows, 1)], sched)
        ctx.launch(lp, spmd)
        ctx.sync()
        ctx.free(lp)
    assert torch.equal(y, z)
