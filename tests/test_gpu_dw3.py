"""The 3x3 / stride-1 depthwise kernel (byte dot products, four channels and columns per
thread) vs the oracle, bit for bit: fewer columns than a group, column groups that overlap,
strips that end inside an image, one and several channel groups, pads 0 to 2, formats of two to
five bits (and a wider filter format), and every form of the epilogue."""
import numpy as np
import pytest

import oracle
from gpuutil import dev, host, log, scalar
from paper_2109_03513_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, H, W, C, pad, activation format, filter format
CASES = [
    (1, 1, 1, 4, 1, (5, 3), (5, 3)),
    (2, 3, 3, 12, 0, (4, 2), (4, 2)),
    (1, 5, 4, 16, 1, (5, 3), (4, 2)),
    (3, 6, 5, 20, 1, (3, 2), (3, 1)),
    (1, 17, 9, 144, 1, (5, 3), (8, 7)),
    (2, 9, 30, 48, 2, (5, 2), (2, 1)),
    (32, 23, 7, 96, 1, (5, 3), (5, 3)),
]


@pytest.mark.parametrize("N,H,W,C,pad,fx,fw", CASES)
@pytest.mark.parametrize("form", ["sums", "y", "relu_y", "codes", "all"])
def test_depthwise3(N, H, W, C, pad, fx, fw, form):
    from paper_2109_03513_amd import esb
    x = wl.random_codes(81, (N, H, W, C), 8)
    w = wl.random_codes(82, (C, 3, 3, 1), 8)
    aX, aW = 0.37, 0.021
    st, oacc, oy = oracle.conv2d(x, w, *fx, aX, *fw, aW, pad=(pad, pad), groups=C)
    assert st == 0
    d = dict(pad=(pad, pad), groups=C)
    head = (dev(x), *fx, scalar(aX), dev(w), *fw, scalar(aW))
    log("depthwise %s %s" % ((N, H, W, C, pad, fx, fw), form))
    if form in ("sums", "y"):
        acc, y = esb.esb_conv2d(*head, want_acc=form == "sums", **d)
        if form == "sums":
            np.testing.assert_array_equal(host(acc), oacc)
        np.testing.assert_array_equal(host(y), oy)
        return
    flat = oy.reshape(-1, C)
    sd = float(np.std(oy)) or 1.0
    qa = np.float32(0.4 * sd)
    r = np.random.default_rng([83, C])
    a = b = res = None
    if form == "all":
        a = r.uniform(-0.5, 1.5, C).astype(np.float32)
        b = (r.standard_normal(C) * 0.3 * sd).astype(np.float32)
        res = (r.standard_normal(oy.shape) * sd).astype(np.float32)
    oz, oc = oracle.post(flat, 5, 3, qa, a=a, bias=b, res=None if res is None else
                         res.reshape(-1, C), relu=True)
    amax = scalar(0.0)
    acc, y, codes = esb.esb_conv2d_post(
        *head, scalar(qa), 5, 3, a=None if a is None else dev(a), b=None if b is None else dev(b),
        residual=None if res is None else dev(res), relu=True, want_acc=form == "all",
        want_y=form != "codes", want_codes=form != "relu_y", absmax=amax, **d)
    if acc is not None:
        np.testing.assert_array_equal(host(acc), oacc)
    if y is not None:
        np.testing.assert_array_equal(host(y).reshape(-1, C).view(np.uint32), oz.view(np.uint32))
    if codes is not None:
        np.testing.assert_array_equal(host(codes).reshape(-1, C), oc)
    assert host(amax)[0] == np.abs(oz).max()
