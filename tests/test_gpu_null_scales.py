"""int32 sums alone need no scales: the calls accept NULL for both, on every contraction kernel
(direct 3x3 with one and several chunks, in halves and with the resident filter; depthwise; short
reductions; tiled, split, decoded once and general), against the oracle's integer sums."""
import numpy as np
import pytest

import oracle
from gpuutil import dev, host, log, torch_cuda
from paper_2109_03513_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, H, W, C, K, R, stride, pad, groups, format
CONVS = [
    (2, 9, 11, 64, 64, 3, 1, 1, 1, (5, 3)),        # direct 3x3, one chunk
    (2, 9, 11, 192, 128, 3, 1, 1, 1, (5, 3)),      # several chunks
    (1, 7, 7, 384, 64, 3, 1, 1, 1, (5, 3)),        # six chunks
    (24, 28, 28, 128, 64, 3, 1, 1, 1, (5, 3)),     # resident filter
    (2, 9, 9, 256, 64, 3, 2, 1, 1, (5, 3)),        # stride 2
    (2, 9, 9, 96, 40, 3, 1, 1, 1, (5, 3)),         # implicit GEMM
    (2, 8, 8, 32, 32, 3, 1, 1, 32, (5, 3)),        # depthwise, C % 16 == 0
    (2, 8, 8, 12, 12, 3, 1, 1, 12, (5, 3)),        # depthwise, C % 4 == 0
    (2, 8, 8, 32, 32, 3, 2, 1, 32, (5, 3)),        # depthwise, stride 2
    (2, 8, 8, 24, 30, 1, 1, 0, 1, (5, 3)),         # 1x1
    (2, 8, 8, 24, 32, 1, 1, 0, 1, (5, 3)),         # 1x1, channels in fours
    (1, 9, 9, 5, 7, 3, 1, 1, 1, (8, 5)),           # general, two int8 planes
]


@pytest.mark.parametrize("N,H,W,C,K,R,st,pad,groups,f", CONVS)
def test_conv_sums_without_scales(N, H, W, C, K, R, st, pad, groups, f):
    from paper_2109_03513_amd import esb
    x = wl.random_codes(61, (N, H, W, C), 8)
    w = wl.random_codes(62, (K, R, R, C // groups), 8)
    d = dict(stride=(st, st), pad=(pad, pad), groups=groups)
    log("sums alone %s" % ((N, H, W, C, K, R, st, pad, groups, f),))
    acc, _ = esb.esb_conv2d(dev(x), *f, None, dev(w), *f, None, want_y=False, **d)
    for img in sorted({0, N - 1}):
        s, oacc, _ = oracle.conv2d(np.ascontiguousarray(x[img:img + 1]), w, *f, 1.0, *f, 1.0, **d)
        assert s == 0
        np.testing.assert_array_equal(host(acc)[img:img + 1], oacc)


@pytest.mark.parametrize("M,N,K,f,ws", [
    (40, 36, 64, (5, 3), False), (300, 200, 512, (5, 3), False), (300, 200, 512, (3, 2), False),
    (50, 30, 33, (5, 3), False), (100, 3000, 4160, (5, 3), True), (1600, 1537, 1152, (5, 3), True)])
def test_gemm_sums_without_scales(M, N, K, f, ws):
    from paper_2109_03513_amd import esb
    torch = torch_cuda()
    A = wl.random_codes(63, (M, K), 8)
    B = wl.random_codes(64, (N, K), 8)
    need = esb.esb_gemm_workspace_size(M, N, K, *f, *f) if ws else 0
    work = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda") if ws else None
    log("sums alone %s" % ((M, N, K, f, ws),))
    acc, _ = esb.esb_gemm(dev(A), *f, None, dev(B), *f, None, want_y=False, workspace=work)
    rows = np.array(sorted({0, 1, M // 2, M - 1}))
    s, oacc, _ = oracle.gemm(np.ascontiguousarray(A[rows]), B, *f, 1.0, *f, 1.0)
    assert s == 0
    np.testing.assert_array_equal(host(acc)[rows], oacc)
