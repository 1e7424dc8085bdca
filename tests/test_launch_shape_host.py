"""Launch shapes that the caller gives in part (teams, units, or a tile): what
the library fills in fits them. Resolved on a host-only context (CPU), and for
choices that need a device, on the GPU.
"""
import ctypes as C

import pytest

from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

_buf = C.create_string_buffer(1 << 21)  # resolving reads no memory: every allocation may be this block
_BASE = (C.addressof(_buf) + 255) // 256 * 256


@U.ALLOC_FN
def _alloc(n, user):
    return _BASE


@U.FREE_FN
def _free(p, user):
    pass


@pytest.fixture(scope="module")
def hctx():
    h = C.c_void_p()
    U.upir_init(U.UPIR_DEVICE_NONE, None, C.byref(h))
    U.upir_set_allocator(h, _alloc, _free, None)
    yield h
    U.upir_finalize(h)


def resolve(h, kind, args, dims, sched=None, spmd=(0, 0), red=None):
    body = U.upir_body(kind, 1, C.cast(C.pointer(args), C.c_void_p), C.sizeof(args))
    L, lp = H.make_loop(dims), C.c_void_p()
    U.upir_loop_parallel(h, C.byref(L), C.byref(sched) if sched else None, C.byref(body),
                         C.byref(red) if red else None, C.byref(lp))
    sp, sc, v, want = U.upir_spmd(), U.upir_sched(), C.c_int32(), H.make_spmd(*spmd)
    U.upir_loop_resolve(h, C.byref(want), lp, C.byref(sp), C.byref(sc), C.byref(v))
    U.upir_loop_free(h, lp)
    return U.VARIANTS[v.value], sp.num_teams, sp.num_units, (sc.tile[0], sc.tile[1])


KINDS = {"f32": U.UPIR_BODY_MATMUL_F32, "bf16": U.UPIR_BODY_MATMUL_BF16, "split": U.UPIR_BODY_MATMUL_SPLIT3}
MMN = [(16, 16, 16), (64, 64, 64), (512, 512, 512), (1000, 1300, 776), (1024, 1024, 1024), (2000, 2000, 2000),
       (4096, 4096, 4096)]


def matmul(h, kind, M, N, K, sched=None, spmd=(0, 0)):
    args = U.upir_matmul_args(0x10000000, 0x20000000, 0x30000000, K, K, N, N, None, 0)
    return resolve(h, KINDS[kind], args, [(0, M, 1), (0, N, 1)], sched, spmd)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("M,N,K", MMN)
def test_matmul_auto_fits_the_units(hctx, kind, M, N, K):
    for teams in (0, 16):
        for units in (0, 256, 512):
            variant, T, Uu, tile = matmul(hctx, kind, M, N, K, None, (teams, units))
            assert variant == "matmul_mfma", (teams, units, tile)
            assert units in (0, Uu) and teams in (0, T)


def test_matmul_tile_for_few_teams(hctx):
    # 16 teams run the 16 tiles of 128 x 128 at once, 64 tiles of 64 x 64 in four rounds
    assert matmul(hctx, "f32", 512, 512, 512, None, (16, 0))[3] == (128, 128)
    assert matmul(hctx, "f32", 512, 512, 512)[3] == (32, 32)


def test_matmul_units_follow_the_chunk(hctx):
    # 576 tiles of 128 x 128: two at a time they are one round of two on 256 units (two teams to a CU), two of two on 512
    tile = (128, 128)
    assert matmul(hctx, "split", 3000, 3000, 3000, H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 2, tile=tile))[2] == 256
    assert matmul(hctx, "split", 3000, 3000, 3000, H.make_sched(U.UPIR_SCHED_STATIC_CHUNK, 2 ** 62, tile=tile))[0] == "matmul_mfma"


@pytest.mark.parametrize("kind", ["bf16", "split"])
def test_matmul_large_tile_on_512_units(hctx, kind):
    for n in (3000, 4096, 8192):
        assert matmul(hctx, kind, n, n, n, None, (0, 512)) == ("matmul_mfma", (-(-n // 256)) ** 2, 512, (256, 256))
        assert matmul(hctx, kind, n, n, n)[2:] == (256, (256, 256))
    # operands over 2 GiB: a named 256 x 256 tile runs on the 512 units that address them, the default is another tile
    big = matmul(hctx, kind, 70000, 512, 16384, H.make_sched(U.UPIR_SCHED_STATIC, tile=(256, 256)))
    assert big[0] == "matmul_mfma" and big[2] == 512
    assert matmul(hctx, kind, 70000, 512, 16384)[3] == (128, 128)


@pytest.mark.parametrize("kind,tile,units", [
    ("f32", (256, 128), {512}), ("f32", (128, 128), {256}), ("f32", (64, 128), {512}), ("f32", (64, 64), {512}),
    ("f32", (32, 32), {512})] + [(k, t, u) for k in ("bf16", "split") for t, u in (
        ((256, 256), {256}), ((128, 128), {256, 512}), ((64, 128), {512}), ((64, 64), {512}), ((32, 32), {512}))])
def test_matmul_units_fit_the_tile(hctx, kind, tile, units):
    for M, N, K in MMN:
        for pol, chunk in ((U.UPIR_SCHED_STATIC, 0), (U.UPIR_SCHED_STATIC_CHUNK, 2)):
            for teams in (0, 16):
                variant, _, Uu, t = matmul(hctx, kind, M, N, K, H.make_sched(pol, chunk, tile=tile), (teams, 0))
                assert variant == "matmul_mfma" and Uu in units and t == tile, (M, N, K, teams)


@pytest.mark.parametrize("pol,chunk", [(U.UPIR_SCHED_AUTO, 0), (U.UPIR_SCHED_STATIC, 0), (U.UPIR_SCHED_STATIC_CHUNK, 1),
                                       (U.UPIR_SCHED_STATIC_CHUNK, 4)])
@pytest.mark.parametrize("n,cols", [(1, 1000), (100, 300), (300, 5000), (1000, 1000), (2500, 80000), (4694, 42607),
                                    (8192, 24414), (16384, 16384), (100000, 256)])
def test_matvec_shape_beside_the_callers(hctx, pol, chunk, n, cols):
    args = U.upir_matvec_args(0x10000000, 0x20000000, 0x30000000, cols, cols)
    shape = lambda spmd: resolve(hctx, U.UPIR_BODY_MATVEC, args, [(0, n, 1)], H.make_sched(pol, chunk), spmd)[1:3]
    for teams in (1, 16, 256, 1024):
        assert shape((teams, 0)) == (teams, 256)
    rest = max(1, min(-(-n // 4), 2048))
    for units in (64, 128, 256, 512, 1024):
        T, Uu = shape((0, units))
        assert Uu == units and T >= rest or (T, Uu) == shape((0, 0))
    if pol != U.UPIR_SCHED_AUTO:
        one = resolve(hctx, U.UPIR_BODY_MATVEC, args, [(0, n, 1)], H.make_sched(pol, chunk, U.UPIR_DIST_UNITS))
        assert one[1:3] == (1, 256)
        assert resolve(hctx, U.UPIR_BODY_MATVEC, args, [(0, n, 1)],
                       H.make_sched(pol, chunk, U.UPIR_DIST_TEAMS))[1] >= rest
    if chunk == 4:  # rows that are not dealt one by one: no eight-wavefront teams
        assert shape((0, 0))[1] < 512


def test_shape_of_a_schedule_from_the_environment(hctx, monkeypatch):
    # the shape beside schedule(runtime) is that beside the schedule it stands for
    S, SC = U.UPIR_SCHED_STATIC, U.UPIR_SCHED_STATIC_CHUNK
    for text, pol, chunk in ((None, S, 0), ("static", S, 0), ("static,1", SC, 1), ("static,2", SC, 2)):
        if text is None:
            monkeypatch.delenv("UPIR_SCHEDULE", raising=False)
        else:
            monkeypatch.setenv("UPIR_SCHEDULE", text)
        for n, cols in ((300, 5000), (8192, 24414), (16384, 16384)):
            args = U.upir_matvec_args(0x10000000, 0x20000000, 0x30000000, cols, cols)
            for dist in (U.UPIR_DIST_TEAMS_UNITS, U.UPIR_DIST_UNITS):
                run, own = (resolve(hctx, U.UPIR_BODY_MATVEC, args, [(0, n, 1)], H.make_sched(p, c, dist))
                            for p, c in ((U.UPIR_SCHED_RUNTIME, 0), (pol, chunk)))
                assert run == own, (text, n, cols, dist)
        for kind in KINDS:
            run, own = (matmul(hctx, kind, 3000, 3000, 3000, H.make_sched(p, c, tile=(128, 128)))
                        for p, c in ((U.UPIR_SCHED_RUNTIME, 0), (pol, chunk)))
            assert run == own, (text, kind)


def test_matvec_short_rows_four_to_a_team(hctx):
    shape = lambda n, cols: resolve(hctx, U.UPIR_BODY_MATVEC, U.upir_matvec_args(
        0x10000000, 0x20000000, 0x30000000, cols, cols), [(0, n, 1)])[1:3]
    assert shape(800, 5000) == (200, 256) and shape(800, 20000) == (800, 64) and shape(512, 5000) == (512, 64)


@pytest.mark.parametrize("pol", [U.UPIR_SCHED_STATIC_CHUNK, U.UPIR_SCHED_DYNAMIC])
def test_stream_units(hctx, pol):
    def units(n, chunk, teams=0, red=None):
        args = U.upir_axpy_args(2.5, 0, 0x10000000, 0x20000000)
        r = H.make_red(red, 0x30000000) if red else None
        return resolve(hctx, U.UPIR_BODY_AXPY, args, [(0, n, 1)], H.make_sched(pol, chunk), (teams, 0), r)[2]
    for n, chunk in ((250003, 64), (250003, 1024), (5000003, 1024)):
        assert units(n, chunk) == units(n, chunk, red=U.UPIR_RED_MAX) == 64  # few ranges, each of them long
        assert units(n, chunk, red=U.UPIR_RED_SUM) == 256                    # the units order the sum
        for teams in (1, 16, 256):
            assert units(n, chunk, teams) == 256
    for n in (1000, 16000, 65000, 250003):  # short ranges
        for chunk in (1, 3, 4, 16):
            assert units(n, chunk) == 256
    assert units(1000003, 16384) == 256 and units(4000, 64) == 256  # a single range on 64 units


@pytest.mark.parametrize("body", ["none", "sync", "async", "filter"])
@pytest.mark.parametrize("N,M", [(34, 66), (500, 500), (1000, 1000), (1500, 2004), (2048, 2048), (3000, 3000),
                                 (4096, 4096), (4832, 5992), (16384, 16384)])
def test_tile_height_beside_the_callers_shape(hctx, body, N, M):
    g = 3 if body == "filter" else 1
    rows, ct = N - 2 * g, -(-(M - 2 * g) // 256)
    any_shape = next((h for h in (128, 64, 32, 16, 8) if (h < 128 or body != "filter") and -(-rows // h) * ct >= 1024), 4)

    def height(spmd):
        dims = [(g, N - g, 1), (g, M - g, 1)]
        if body == "filter":
            args = U.upir_filter7_args(0x10000000, 0x7000000000, 0x9000, M)
            return resolve(hctx, U.UPIR_BODY_FILTER7, args, dims, None, spmd)[3][0]
        red = None if body == "none" else H.make_red(U.UPIR_RED_MAX, 0x9000, async_=body == "async")
        args = U.upir_jacobi5_args(0x10000000, 0x7000000000, M)
        return resolve(hctx, U.UPIR_BODY_JACOBI5, args, dims, None, spmd, red)[3][0]

    free = height((0, 0))
    assert height((0, 256)) == free
    for teams in (1, 256, 1024):
        assert height((teams, 0)) == height((teams, 256)) == any_shape
    for units in (64, 128):
        assert height((0, units)) == min(free, any_shape)
    for units in (512, 1024):
        assert height((0, units)) == max(free, any_shape)
    assert height((0, 100)) == any_shape


@pytest.mark.parametrize("N,M", [(4096, 4096), (8192, 8192), (8300, 8300), (11600, 11600), (16384, 16384),
                                 (23000, 23000), (600000, 12), (12, 600000), (1200000, 300)])
def test_async_partials_fit_the_first_fold_buffers(hctx, N, M):
    # one partial per wavefront; the buffers hold 65,536, or what a tiling of 128 rows throughout would need
    tiles = -(-(N - 2) // 128) * -(-(M - 2) // 256)
    red = H.make_red(U.UPIR_RED_MAX, 0x9000, async_=True)
    args = U.upir_jacobi5_args(0x10000000, 0x7000000000, M)
    _, T, Uu, _ = resolve(hctx, U.UPIR_BODY_JACOBI5, args, [(1, N - 1, 1), (1, M - 1, 1)], None, (0, 0), red)
    assert T * Uu // 64 <= max(65536, 4 * tiles)


@pytest.mark.gpu
def test_async_memory():
    # what the first async reduction of a context asks the allocator for
    torch = pytest.importorskip("torch")
    sizes = []

    @U.ALLOC_FN
    def alloc(n, user):
        sizes.append(n)
        return torch.cuda.caching_allocator_alloc(n)

    @U.FREE_FN
    def free(p, user):
        torch.cuda.caching_allocator_delete(p)

    h = C.c_void_p()
    x = torch.rand(1000, device="cuda")
    r = torch.zeros(1, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    U.upir_init(0, None, C.byref(h))
    U.upir_set_allocator(h, alloc, free, None)
    args = U.upir_sum_args(x.data_ptr(), U.UPIR_DT_F32, 0)
    body = U.upir_body(U.UPIR_BODY_SUM, 1, C.cast(C.pointer(args), C.c_void_p), C.sizeof(args))
    L, lp, red = H.make_loop([(0, 1000, 1)]), C.c_void_p(), H.make_red(U.UPIR_RED_MAX, r.data_ptr(), async_=True)
    U.upir_loop_parallel(h, C.byref(L), None, C.byref(body), C.byref(red), C.byref(lp))
    made = sum(sizes)
    U.upir_spmd_launch(h, None, (C.c_void_p * 1)(lp.value), 1)
    U.upir_sync(h)
    assert r.item() == float(x.max())
    assert sum(sizes) - made <= 2 * 65536 * 8
    U.upir_finalize(h)


@pytest.mark.gpu
def test_matmul_tuned_choice_fits_the_units():
    torch = pytest.importorskip("torch")
    n = 512
    A, Cm = torch.rand(n, n, device="cuda"), torch.zeros(n, n, device="cuda")
    with H.Context(0) as ctx:
        args = U.upir_matmul_args(A.data_ptr(), A.data_ptr(), Cm.data_ptr(), n, n, n, n, None, 0)
        lp = ctx.loop(U.UPIR_BODY_MATMUL_BF16, args, [(0, n, 1), (0, n, 1)])
        U.upir_tune(ctx.h, None, lp, 3, None, None, None)
        for units in (0, 256, 512):
            sp, sc, v = ctx.resolve(lp, H.make_spmd(0, units))
            assert U.VARIANTS[v] == "matmul_mfma" and units in (0, sp.num_units), (units, sp.num_units, sc.tile[0])
        ctx.free(lp)
