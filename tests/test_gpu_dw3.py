"""The 3x3 / stride-1 depthwise kernel (byte dot products, four channels and columns per
thread) vs the oracle, bit for bit: fewer columns than a group, column groups that overlap,
strips that end inside an image, one and several channel groups, pads 0 to 2, formats of two to
five bits (and a wider filter format), every form of the epilogue, strips of 4, 8 and 16 rows, and
both sides of the lines between it and the other depthwise kernels."""
import numpy as np
import pytest

import oracle
from gpuutil import dev, host, log, scalar, torch_cuda
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


def check_images(N, H, W, C, form, images, seed, f=(5, 3), fw=(5, 3), pad=1):
    """One form of a 3x3 layer on N images, the listed ones against the oracle."""
    from paper_2109_03513_amd import esb
    x = wl.random_codes(seed, (N, H, W, C), 8)
    w = wl.random_codes(seed + 1, (C, 3, 3, 1), 8)
    d = dict(pad=(pad, pad), groups=C)
    xs = np.ascontiguousarray(x[images])
    st, oacc, oy = oracle.conv2d(xs, w, *f, 0.37, *fw, 0.021, **d)
    assert st == 0
    log("depthwise %s %s" % ((N, H, W, C, f, fw, pad), form))
    head = (dev(x), *f, scalar(0.37), dev(w), *fw, scalar(0.021))
    if form in ("y", "sums"):
        acc, y = esb.esb_conv2d(*head, want_acc=form == "sums", **d)
        if form == "sums":
            np.testing.assert_array_equal(host(acc)[images], oacc)
        np.testing.assert_array_equal(host(y)[images], oy)
        return
    sd = float(np.std(oy)) or 1.0
    qa = np.float32(0.4 * sd)
    r = np.random.default_rng([seed, C])
    a = b = res = None
    if form == "all":
        a = r.uniform(-0.5, 1.5, C).astype(np.float32)
        b = (r.standard_normal(C) * 0.3 * sd).astype(np.float32)
    if form in ("all", "residual"):
        res = (r.standard_normal((N,) + oy.shape[1:]) * sd).astype(np.float32)
    oz, oc = oracle.post(oy.reshape(-1, C), 5, 3, qa, a=a, bias=b, relu=True,
                         res=None if res is None else res[images].reshape(-1, C))
    amax = scalar(0.0)
    _, y, codes = esb.esb_conv2d_post(
        *head, scalar(qa), 5, 3, a=None if a is None else dev(a), b=None if b is None else dev(b),
        residual=None if res is None else dev(res), relu=True, want_codes=form in ("codes", "all"),
        want_y=form != "codes", absmax=amax, **d)
    if y is not None:
        np.testing.assert_array_equal(host(y)[images].reshape(-1, C).view(np.uint32), oz.view(np.uint32))
        assert host(amax)[0] == np.abs(host(y)).max()
    if codes is not None:
        np.testing.assert_array_equal(host(codes)[images].reshape(-1, C), oc)


@pytest.mark.parametrize("rows", [4, 8, 16])
@pytest.mark.parametrize("form", ["y", "relu_y", "codes", "sums", "all"])
def test_strip_heights(rows, form):
    """Strips of that many rows (57 output rows in strips of 4, 8 and 15), 58 columns."""
    H, W, C = 57, 58, 192
    cus = torch_cuda().cuda.get_device_properties(0).multi_processor_count
    want = cus * 8 * 64                                     # threads that fill the chip
    per_image = -(-W // 4) * (C // 4)
    N = -(-want // (per_image * -(-H // rows)))             # the fewest images that take this height
    assert per_image * N * -(-H // rows) >= want
    assert rows == 16 or per_image * N * -(-H // (2 * rows)) < want
    check_images(N, H, W, C, form, [0, N // 2, N - 1], 84)


@pytest.mark.parametrize("N,H,W,C", [
    (1, 9, 9, 60), (1, 9, 9, 64), (1, 9, 9, 16), (1, 9, 9, 12), (1, 9, 9, 176), (1, 9, 9, 192),
    (16, 64, 64, 4), (15, 64, 64, 4), (32, 64, 64, 4), (64, 64, 64, 4),
    (4, 1, 1, 16), (4, 1, 1, 48), (3, 3, 3, 48), (3, 3, 3, 32), (100, 3, 3, 20),
    (46, 1, 1, 64), (47, 1, 1, 64), (2083, 1, 1, 144), (2084, 1, 1, 144), (3472, 1, 1, 144), (3473, 1, 1, 144),
    (5, 1, 1, 100), (3000, 1, 1, 100), (3, 2, 2, 32), (82, 2, 2, 100), (81, 2, 2, 100), (3641, 2, 2, 36),
    (3640, 2, 2, 36), (1619, 3, 3, 36), (1618, 3, 3, 36), (3237, 3, 3, 36), (3236, 3, 3, 36)])
@pytest.mark.parametrize("form", ["y", "relu_y", "codes", "sums", "residual", "all"])
def test_routes(N, H, W, C, form):
    check_images(N, H, W, C, form, sorted({0, N // 2, N - 1}), 86)


@pytest.mark.parametrize("f,fw,pad", [((5, 2), (2, 1), 2), ((4, 2), (4, 2), 0), ((4, 3), (5, 3), 1),
                                      ((3, 2), (3, 1), 1), ((2, 1), (8, 7), 1)])
@pytest.mark.parametrize("form", ["y", "relu_y", "codes", "sums", "residual", "all"])
def test_formats(f, fw, pad, form):
    check_images(2, 7, 10, 192, form, [0, 1], 88, f, fw, pad)
