"""The short-reduction kernel (1x1 convolutions, GEMMs with K <= 256) vs the oracle, bit for
bit: reductions at the edges of its 64-byte steps and of both load widths, rows and channels
that fill no tile, strided pixels, row pitches beyond K, several channel shares per tile row,
and every form of the epilogue."""
import ctypes

import numpy as np
import pytest

import oracle
from gpuutil import dev, host, log, scalar, torch_cuda
from paper_2109_03513_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, H, W, C, K, stride, activation format, filter format
CONVS = [
    (1, 1, 1, 8, 1, 1, (5, 3), (5, 3)),
    (1, 7, 5, 24, 30, 1, (5, 3), (5, 3)),
    (2, 13, 9, 24, 144, 1, (5, 3), (4, 2)),
    (1, 9, 9, 64, 64, 2, (4, 2), (4, 2)),
    (3, 6, 7, 72, 33, 1, (3, 2), (3, 1)),
    (2, 11, 8, 144, 24, 1, (5, 3), (5, 3)),
    (1, 8, 8, 200, 100, 2, (6, 4), (5, 2)),
    (1, 5, 7, 256, 1024, 1, (5, 3), (5, 3)),
    (70, 30, 30, 16, 32, 1, (5, 3), (5, 3)),     # one tile for most waves, none for some
    (1, 40, 40, 24, 24, 1, (5, 3), (5, 3)),
]


@pytest.mark.parametrize("N,H,W,C,K,st,fx,fw", CONVS)
@pytest.mark.parametrize("form", ["sums", "y", "relu_y", "residual", "codes", "all"])
def test_conv1x1(N, H, W, C, K, st, fx, fw, form):
    from paper_2109_03513_amd import esb
    x = wl.random_codes(91, (N, H, W, C), 8)
    w = wl.random_codes(92, (K, 1, 1, C), 8)
    aX, aW = 0.37, 0.021
    s, oacc, oy = oracle.conv2d(x, w, *fx, aX, *fw, aW, stride=(st, st))
    assert s == 0
    head = (dev(x), *fx, scalar(aX), dev(w), *fw, scalar(aW))
    log("conv1x1 %s %s" % ((N, H, W, C, K, st, fx, fw), form))
    if form in ("sums", "y"):
        acc, y = esb.esb_conv2d(*head, want_acc=form == "sums", stride=(st, st))
        if form == "sums":
            np.testing.assert_array_equal(host(acc), oacc)
        np.testing.assert_array_equal(host(y), oy)
        return
    sd = float(np.std(oy)) or 1.0
    qa = np.float32(0.4 * sd)
    r = np.random.default_rng([93, C, K])
    a = b = res = None
    if form == "all":
        a = r.uniform(-0.5, 1.5, K).astype(np.float32)
        b = (r.standard_normal(K) * 0.3 * sd).astype(np.float32)
    if form in ("all", "residual"):
        res = (r.standard_normal(oy.shape) * sd).astype(np.float32)
    relu = form != "residual"
    oz, oc = oracle.post(oy.reshape(-1, K), 5, 3, qa, a=a, bias=b,
                         res=None if res is None else res.reshape(-1, K), relu=relu)
    amax = scalar(0.0)
    acc, y, codes = esb.esb_conv2d_post(
        *head, scalar(qa), 5, 3, a=None if a is None else dev(a), b=None if b is None else dev(b),
        residual=None if res is None else dev(res), relu=relu, want_acc=form == "all",
        want_y=form != "codes", want_codes=form in ("codes", "all"), absmax=amax, stride=(st, st))
    if acc is not None:
        np.testing.assert_array_equal(host(acc), oacc)
    if y is not None:
        np.testing.assert_array_equal(host(y).reshape(-1, K).view(np.uint32), oz.view(np.uint32))
    if codes is not None:
        np.testing.assert_array_equal(host(codes).reshape(-1, K), oc)
    assert host(amax)[0] == np.abs(oz).max()


@pytest.mark.parametrize("M,N,K,lda,ldb,ldc,off", [
    (100, 70, 48, 64, 56, 72, 0), (33, 20, 96, 104, 96, 23, 8), (65, 40, 120, 120, 128, 40, 0),
    (1, 1, 16, 16, 16, 1, 0)])
def test_gemm_row_pitches(M, N, K, lda, ldb, ldc, off):
    """Operands and outputs with row pitches of their own and bases at 8 bytes."""
    from paper_2109_03513_amd import esb
    torch = pytest.importorskip("torch")
    A = wl.random_codes(94, (M, lda), 8)
    B = wl.random_codes(95, (N, ldb), 8)
    st, oacc, oy = oracle.gemm(np.ascontiguousarray(A[:, :K]), np.ascontiguousarray(B[:, :K]),
                               5, 3, 0.37, 5, 3, 0.021)
    assert st == 0
    dA = torch.zeros(M * lda + 16, dtype=torch.uint8, device="cuda")[off:off + M * lda]
    dB = torch.zeros(N * ldb + 16, dtype=torch.uint8, device="cuda")[off:off + N * ldb]
    dA.copy_(dev(A).reshape(-1))
    dB.copy_(dev(B).reshape(-1))
    acc = torch.full((M, ldc), -7, dtype=torch.int32, device="cuda")
    y = torch.full((M, ldc), -7.0, dtype=torch.float32, device="cuda")
    a, b = scalar(0.37), scalar(0.021)
    P = lambda t: ctypes.c_void_p(t.data_ptr())   # noqa: E731
    for want in ((acc, y), (None, y)):
        y.fill_(-7.0)
        esb._check("esb_gemm", esb.lib().esb_gemm(
            M, N, K, P(dA), lda, 5, 3, P(a), P(dB), ldb, 5, 3, P(b), 0,
            None if want[0] is None else P(acc), P(y), ldc, esb._stream(None)))
        np.testing.assert_array_equal(host(y)[:, :N], oy)
        assert (host(y)[:, N:] == -7.0).all()
    np.testing.assert_array_equal(host(acc)[:, :N], oacc)
    assert (host(acc)[:, N:] == -7).all()


def rows_per_wave(gy):
    """Rows that give every wave of a launch with gy channel shares one tile."""
    return 32 * 4 * -(-4 * torch_cuda().cuda.get_device_properties(0).multi_processor_count // gy)


@pytest.mark.parametrize("N,K,gy", [(32, 16, 1), (1024, 256, 5)])
@pytest.mark.parametrize("form", ["sums", "y", "residual", "codes"])
def test_several_tiles_per_wave(N, K, gy, form):
    """More than twice as many tiles as waves, the last one ragged: the next tile's codes and
    residual are fetched while this one is computed, the maximum runs over all tiles."""
    from paper_2109_03513_amd import esb
    M = 2 * rows_per_wave(gy) + 32 * 5 + 7
    A = wl.random_codes(96, (M, K), 8)
    B = wl.random_codes(97, (N, K), 8)
    step = 1 if M * N * K < 2 ** 28 else 97
    rows = np.unique(np.concatenate([np.arange(0, M, step), np.arange(M - 40, M)]))
    st, oacc, oy = oracle.gemm(np.ascontiguousarray(A[rows]), B, 5, 3, 0.37, 5, 3, 0.021)
    assert st == 0
    log("several tiles per wave %s %s" % ((M, N, K), form))
    head = (dev(A), 5, 3, scalar(0.37), dev(B), 5, 3, scalar(0.021))
    if form in ("sums", "y"):
        acc, y = esb.esb_gemm(*head, want_acc=form == "sums")
        if form == "sums":
            np.testing.assert_array_equal(host(acc)[rows], oacc)
        np.testing.assert_array_equal(host(y)[rows], oy)
        return
    sd = float(np.std(oy))
    qa = np.float32(0.4 * sd)
    torch = torch_cuda()
    res = torch.randn(M, N, device="cuda", generator=torch.Generator("cuda").manual_seed(3)) * sd
    ores = host(res)[rows] if form == "residual" else None
    oz, oc = oracle.post(oy, 5, 3, qa, res=ores, relu=form == "codes")
    amax = scalar(0.0)
    _, y, codes = esb.esb_gemm_post(*head, scalar(qa), 5, 3, residual=res if form == "residual" else None,
                                    relu=form == "codes", want_codes=form == "codes",
                                    want_y=form == "residual", absmax=amax)
    if form == "codes":
        np.testing.assert_array_equal(host(codes)[rows], oc)
        _, y, _ = esb.esb_gemm_post(*head, scalar(qa), 5, 3, relu=True, want_codes=False, want_y=True)
    np.testing.assert_array_equal(host(y)[rows].view(np.uint32), oz.view(np.uint32))
    assert host(amax)[0] == np.abs(host(y)).max()


# M, N, K on both sides of the lines between this kernel and the tiled and general ones
ROUTES = [
    (7, 24, 64), (8, 24, 64), (7, 8, 64), (5, 16, 200), (40, 31, 48), (40, 32, 48), (31, 9, 64), (33, 9, 64),
    (2344, 65, 256), (2343, 65, 256), (100, 40, 8), (3000, 200, 8), (3001, 200, 8), (700, 33, 128),
    (20000, 36, 64), (19999, 36, 64), (46000, 32, 256), (1200, 1000, 96), (1203, 1001, 200),
    (2500, 400, 24), (2499, 400, 24), (11719, 256, 64), (11718, 256, 64), (15000, 400, 8), (14999, 400, 8),
    (50000, 64, 24), (50000, 50, 24), (50000, 50, 8)]


@pytest.mark.parametrize("M,N,K", ROUTES)
@pytest.mark.parametrize("form", ["sums", "acc", "affine_codes", "affine_all", "residual", "codes", "sums_all"])
def test_routes(M, N, K, form):
    from paper_2109_03513_amd import esb
    A = wl.random_codes(98, (M, K), 8)
    B = wl.random_codes(99, (N, K), 8)
    rows = np.unique(np.concatenate([np.arange(0, M, max(1, M // 300)), np.arange(max(0, M - 33), M)]))
    st, oacc, oy = oracle.gemm(np.ascontiguousarray(A[rows]), B, 5, 3, 0.37, 5, 3, 0.021)
    assert st == 0
    log("routes %s %s" % ((M, N, K), form))
    head = (dev(A), 5, 3, scalar(0.37), dev(B), 5, 3, scalar(0.021))
    if form in ("sums", "acc"):
        acc, y = esb.esb_gemm(*head, want_y=form == "sums")
        np.testing.assert_array_equal(host(acc)[rows], oacc)
        if y is not None:
            np.testing.assert_array_equal(host(y)[rows], oy)
        return
    r = np.random.default_rng([98, N, K])
    sd = float(np.std(oy)) or 1.0
    qa = np.float32(0.4 * sd)
    a = b = res = None
    if form != "codes":
        a = r.uniform(-0.5, 1.5, N).astype(np.float32)
        b = (r.standard_normal(N) * 0.3 * sd).astype(np.float32)
    if form == "residual":
        a = b = None
        res = (r.standard_normal((M, N)) * sd).astype(np.float32)
    codes_only, y_only = form in ("codes", "affine_codes"), form == "residual"
    oz, oc = oracle.post(oy, 5, 3, qa, a=a, bias=b, res=None if res is None else res[rows], relu=True)
    acc, y, codes = esb.esb_gemm_post(
        *head, scalar(qa), 5, 3, a=None if a is None else dev(a), b=None if b is None else dev(b),
        residual=None if res is None else dev(res), relu=True, want_codes=not y_only,
        want_y=not codes_only, want_acc=form == "sums_all")
    if acc is not None:
        np.testing.assert_array_equal(host(acc)[rows], oacc)
    if y is not None:
        np.testing.assert_array_equal(host(y)[rows].view(np.uint32), oz.view(np.uint32))
    if codes is not None:
        np.testing.assert_array_equal(host(codes)[rows], oc)
