"""GPU parity of the matmul tiles at sizes where their edges can go wrong:
fewer rows, columns or k than a tile, a vector of four or a k step; partial
vectors at the last column and k; operands that start off a 16-byte boundary
and pitches that are no multiple of four; several tiles per team.

Integer matrices with entries in {-2..2} make every product and partial sum
exact, so the comparison is exact in all precisions (bfloat16 holds these
entries, the split's low parts are zero).
"""
import numpy as np
import pytest

from oracle import bodies
from paper_2209_10643_amd import helpers as H
from paper_2209_10643_amd import upir as U

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KINDS = {"f32": U.UPIR_BODY_MATMUL_F32, "bf16": U.UPIR_BODY_MATMUL_BF16, "split": U.UPIR_BODY_MATMUL_SPLIT3}


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


def placed(a, off, pad):
    """Device copy of `a` whose rows are `pad` longer and which starts `off`
    elements into its buffer; NaN around it."""
    r, c = a.shape
    buf = torch.full((off + r * (c + pad) + 4,), float("nan"), device="cuda")
    buf[off:off + r * (c + pad)].view(r, c + pad)[:, :c] = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return buf, buf.data_ptr() + 4 * off, c + pad


def product(ctx, kind, A, B, sched=None, spmd=None, off=0, pad=0):
    M, K = A.shape
    N = B.shape[1]
    ta, pa, lda = placed(A, off, pad)
    tb, pb, ldb = placed(B, off, pad)
    tc = torch.full((M * (N + pad) + 8,), -7.0, device="cuda")
    args = U.upir_matmul_args(pa, pb, tc.data_ptr() + 4 * off, K, lda, ldb, N + pad, None, 0)
    lp = ctx.loop(KINDS[kind], args, [(0, M, 1), (0, N, 1)], sched)
    ctx.launch(lp, spmd)
    ctx.sync()
    ctx.free(lp)
    out = tc.cpu().numpy()
    box = out[off:off + M * (N + pad)].reshape(M, N + pad)
    assert (out[:off] == -7.0).all() and (box[:, N:] == -7.0).all() and (out[off + M * (N + pad):] == -7.0).all()
    return box[:, :N]


SHAPES = [(1, 1, 1), (5, 3, 2), (31, 33, 7), (33, 31, 64), (65, 66, 63), (64, 64, 128), (100, 130, 129), (130, 67, 321)]


@pytest.mark.parametrize("tile,units", [((32, 32), 512), ((64, 64), 512), ((64, 128), 512), ((128, 128), 256),
                                        ((256, 128), 512), (None, 0)])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_f32_tiles(ctx, tile, units, M, N, K):
    print(f"f32 {M}x{N}x{K} tile={tile}", flush=True)
    rng = np.random.default_rng(M * N + K)
    A, B = (rng.integers(-2, 3, s).astype(np.float32) for s in ((M, K), (K, N)))
    want = bodies.matmul(A, B)
    for off, pad, sched, teams in ((0, 0, U.UPIR_SCHED_STATIC, 0), (1, 3, U.UPIR_SCHED_STATIC, 2),
                                   (3, 2, U.UPIR_SCHED_STATIC_CHUNK, 3)):
        s = H.make_sched(sched, 1 if sched == U.UPIR_SCHED_STATIC_CHUNK else 0, tile=tile) if tile else None
        got = product(ctx, "f32", A, B, s, H.make_spmd(teams, units), off, pad)
        assert np.array_equal(got.astype(np.float64), want), (off, pad)


@pytest.mark.parametrize("kind", ["bf16", "split"])
@pytest.mark.parametrize("tile,units", [((32, 32), 512), ((64, 64), 512), ((64, 128), 512), ((128, 128), 512),
                                        ((128, 128), 256),
                                        ((256, 256), 256), ((256, 256), 512), ((16, 16), 64), (None, 0)])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_bf16_tiles(ctx, kind, tile, units, M, N, K):
    """The tiles that read float32 operands themselves, those behind the
    pre-pass (K no multiple of eight: the workspace's last chunk of k is
    padded) and the schedule-exact kernel."""
    print(f"{kind} {M}x{N}x{K} tile={tile} units={units}", flush=True)
    rng = np.random.default_rng(M * N + K)
    A, B = (rng.integers(-2, 3, s).astype(np.float32) for s in ((M, K), (K, N)))
    want = bodies.matmul(A, B)
    for off, pad, teams in ((0, 0, 0), (1, 3, 2)):
        s = H.make_sched(U.UPIR_SCHED_STATIC, tile=tile) if tile else None
        got = product(ctx, kind, A, B, s, H.make_spmd(teams, units), off, pad)
        assert np.array_equal(got.astype(np.float64), want), (off, pad)


@pytest.mark.parametrize("units", [256, 512])
def test_split_keeps_its_low_parts(ctx, units):
    """1 + 2^-9 has a low part: the product of the rounded operands alone is
    off by 2^-8 of each entry."""
    M, N, K = 70, 66, 45
    A, B = np.full((M, K), 1 + 2.0 ** -9, np.float32), np.ones((K, N), np.float32)
    B[::2] = -(1 + 2.0 ** -9)
    for tile in ((128, 128),) + (((64, 64), (32, 32)) if units == 512 else ((256, 256),)):
        got = product(ctx, "split", A, B, H.make_sched(U.UPIR_SCHED_STATIC, tile=tile), H.make_spmd(0, units))
        assert bodies.frob_rel(got, bodies.matmul_split3(A, B)) <= 1e-5


def test_pending_fold_before_an_unaligned_product(ctx):
    """An async sum's fold is pending when a product that takes no fold along
    runs: the sum is delivered, the product is right."""
    n, M, N, K = 5000, 70, 45, 33
    x = torch.ones(n, device="cuda")
    r = torch.zeros(1, dtype=torch.float64, device="cuda")
    lp = ctx.loop(U.UPIR_BODY_SUM, U.upir_sum_args(x.data_ptr(), U.UPIR_DT_F32, 0), [(0, n, 1)], None,
                  H.make_red(U.UPIR_RED_SUM, r.data_ptr(), async_=True))
    ctx.launch(lp)
    rng = np.random.default_rng(3)
    A, B = (rng.integers(-2, 3, s).astype(np.float32) for s in ((M, K), (K, N)))
    got = product(ctx, "f32", A, B)
    assert np.array_equal(got.astype(np.float64), bodies.matmul(A, B))
    assert r.item() == n
    ctx.free(lp)
