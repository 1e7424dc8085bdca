"""Chunks far longer than the loop, up to the largest the ABI takes: the same as
one chunk of the whole loop. On the CPU the arithmetic against 128-bit
integers; on the GPU every policy that takes a chunk, on launch shapes whose
products with the chunk pass 64 bits.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

import synth
from oracle import bodies
from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHUNKS = [10 ** 15, 2 ** 62, 2 ** 63 - 1]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_chunk_arithmetic(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-fsanitize=undefined",
                        "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2209_10643_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "chunk_math_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


@pytest.fixture(scope="module")
def ctx():
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    U.lib()
    s = torch.cuda.Stream()
    prev = torch.cuda.current_stream()
    torch.cuda.set_stream(s)
    c = H.Context(0, stream=s)
    yield c
    c.close()
    torch.cuda.set_stream(prev)


SHAPES = [(0, 0), (1, 64), (1000, 512), (7, 1000)]


@pytest.mark.gpu
@pytest.mark.parametrize("chunk", CHUNKS)
@pytest.mark.parametrize("pol,dist", [(U.UPIR_SCHED_STATIC_CHUNK, U.UPIR_DIST_TEAMS_UNITS),
                                      (U.UPIR_SCHED_STATIC_CHUNK, U.UPIR_DIST_TEAMS),
                                      (U.UPIR_SCHED_STATIC_CHUNK, U.UPIR_DIST_UNITS),
                                      (U.UPIR_SCHED_DYNAMIC, 0), (U.UPIR_SCHED_GUIDED, 0)])
def test_every_iteration_once(ctx, pol, dist, chunk):
    import torch
    for n in (0, 1, 4097):
        for step in (1, -2):
            for T, Uu in SHAPES:
                T = min(T, 1) if dist == U.UPIR_DIST_UNITS else T
                print(f"cover n={n} step={step} pol={pol} dist={dist} chunk={chunk} T={T} U={Uu}", flush=True)
                cnt = torch.zeros(max(n, 1) + 64, dtype=torch.int32, device="cuda")
                lb = 2 * n if step < 0 else 0
                lp = ctx.loop(U.UPIR_BODY_COVER, U.upir_cover_args(cnt.data_ptr()), [(lb, lb + n * step, step)],
                              H.make_sched(pol, chunk, dist))
                for _ in range(2):
                    ctx.launch(lp, H.make_spmd(T, Uu))
                ctx.sync()
                ctx.free(lp)
                got = cnt.cpu().numpy()
                assert (got[:n] == 2).all() and (got[n:] == 0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("chunk", CHUNKS)
def test_tiles_and_rows(ctx, chunk):
    import torch
    N, M = 70, 515
    u = synth.uniform_01(81, 0, N * M).reshape(N, M)
    want, res = bodies.jacobi5(u, 1)
    A, x = synth.uniform_pm1(81, 1, 300 * 257).reshape(300, 257), synth.uniform_pm1(81, 2, 257)
    for T, Uu in ((0, 0), (5, 64), (1000, 512)):
        print(f"tiles chunk={chunk} T={T} U={Uu}", flush=True)
        a, b = torch.from_numpy(u).cuda(), torch.from_numpy(u).cuda()
        r = torch.zeros(1, dtype=torch.float64, device="cuda")
        for tile in ((8, 256), (4, 16)):
            lp = ctx.loop(U.UPIR_BODY_JACOBI5, U.upir_jacobi5_args(a.data_ptr(), b.data_ptr(), M),
                          [(1, N - 1, 1), (1, M - 1, 1)], H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, chunk, tile=tile),
                          H.make_red(U.UPIR_RED_MAX, r.data_ptr()))
            ctx.launch(lp, H.make_spmd(T, Uu))
            ctx.sync()
            ctx.free(lp)
            assert np.array_equal(b.cpu().numpy(), want) and r.item() == res[0]
        w = torch.ones(49, device="cuda")
        f = torch.zeros(N, M, device="cuda")
        lp = ctx.loop(U.UPIR_BODY_FILTER7, U.upir_filter7_args(a.data_ptr(), f.data_ptr(), w.data_ptr(), M),
                      [(3, N - 3, 1), (3, M - 3, 1)], H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, chunk, tile=(8, 256)))
        ctx.launch(lp, H.make_spmd(T, Uu))
        ctx.sync()
        ctx.free(lp)
        assert np.array_equal(f.cpu().numpy()[3:-3, 3:-3], bodies.filter7(u, np.ones((7, 7), np.float32))[3:-3, 3:-3])
        tA, tx, ty = torch.from_numpy(A).cuda(), torch.from_numpy(x).cuda(), torch.zeros(300, device="cuda")
        lp = ctx.loop(U.UPIR_BODY_MATVEC, U.upir_matvec_args(tA.data_ptr(), tx.data_ptr(), ty.data_ptr(), 257, 257),
                      [(0, 300, 1)], H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, chunk))
        ctx.launch(lp, H.make_spmd(T, Uu))
        ctx.sync()
        ctx.free(lp)
        assert bodies.frob_rel(ty.cpu().numpy(), bodies.matvec(A, x)) <= 1e-5
        B = synth.int_range(81, 3, 130 * 70, -2, 3).astype(np.float32).reshape(130, 70)
        tB, tC = torch.from_numpy(B).cuda(), torch.zeros(130, 130, device="cuda")
        Bt = torch.from_numpy(np.ascontiguousarray(B.T)).cuda()
        for kind in (U.UPIR_BODY_MATMUL_F32, U.UPIR_BODY_MATMUL_BF16):
            for tile in ((64, 64), (128, 128), (16, 16)):
                lp = ctx.loop(kind, U.upir_matmul_args(tB.data_ptr(), Bt.data_ptr(), tC.data_ptr(), 70, 70, 130, 130, None, 0),
                              [(0, 130, 1), (0, 130, 1)], H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, chunk, tile=tile))
                ctx.launch(lp, H.make_spmd(T, Uu))
                ctx.sync()
                ctx.free(lp)
                assert np.array_equal(tC.cpu().numpy(), B @ B.T)
