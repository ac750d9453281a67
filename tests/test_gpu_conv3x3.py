"""The direct 3x3 / pad-1 convolution kernels, stride 1 and 2 (input and output channels in
multiples of 64 on the fp8 MFMA; tiles of 256, 128 or 64 output pixels over the batch,
crossing image boundaries; input channels in chunks of 64; the filter slice per chunk, or
resident for the workgroup; with stride 2 the even padded columns of a patch row first)
against the oracle's convolution
and post-processing: bit-exact int32 sums, fp32 outputs and codes, equal running maximum;
and bit for bit equal to the implicit-GEMM path, which an input one byte off a 16-byte
boundary takes."""
import numpy as np
import pytest

import oracle
from gpuutil import dev, host, log, scalar, torch_cuda
from paper_2109_03513_amd import workloads as wl

pytestmark = pytest.mark.gpu
ALPHA_X, ALPHA_W = 0.43, 0.027


@pytest.fixture(scope="module")
def esb():
    from paper_2109_03513_amd import esb as e
    e.lib()
    return e


def unaligned(torch, a):
    """A device copy of the uint8 array a whose data starts one byte past a 16-byte boundary."""
    buf = torch.empty(a.size + 16, dtype=torch.uint8, device="cuda")
    v = buf[1:1 + a.size].view(a.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    assert v.data_ptr() % 16 == 1
    return v


CASES = [
    # N, H, W, C, K, fx, fw, variant
    (2, 56, 56, 64, 64, (5, 3), (5, 3), "plain"),     # the ResNet18 l1 shape, batch 2
    (3, 7, 7, 64, 64, (5, 3), (5, 3), "all"),         # 49-pixel images: 64-pixel tiles over two
    (1, 13, 5, 64, 64, (4, 2), (5, 3), "relu"),       # H != W, ragged last tile, mixed formats
    (2, 9, 62, 64, 64, (5, 3), (4, 2), "residual"),   # widest rows taken (Q + 2 = 64)
    (1, 1, 1, 64, 64, (5, 3), (5, 3), "affine"),      # one pixel
    (4, 17, 23, 64, 64, (6, 3), (4, 1), "all"),       # ESB(6,3) x ESB(4,1)
    # several chunks of input channels and / or tiles of output channels
    (2, 28, 28, 128, 128, (5, 3), (5, 3), "all"),     # the l2 shape, batch 2 (1568 pixels)
    (3, 14, 14, 256, 192, (5, 3), (4, 2), "relu"),    # four chunks, three channel tiles
    (1, 5, 9, 192, 64, (5, 3), (5, 3), "residual"),   # three chunks, ragged
    (2, 7, 7, 512, 128, (5, 3), (5, 3), "plain"),     # eight chunks (the l4 reduction)
    # one chunk (all of this list): 64-pixel tiles, for tiles of 128 give fewer workgroups than
    # CUs (the larger tiles: test_conv3x3_one_chunk); several chunks: 128-pixel tiles down to
    # half a workgroup per CU
    (50, 7, 7, 128, 512, (5, 3), (5, 3), "plain"),    # several chunks, 128-pixel tiles
    (16, 14, 14, 64, 512, (5, 3), (5, 3), "affine"),  # one chunk, eight channel tiles
    (8, 1, 40, 128, 64, (5, 3), (5, 3), "all"),       # several chunks, 64-pixel tiles (one-row
                                                      # images: 128 pixels need 15 patch rows)
    # several chunks and more than 16384 pixels: the resident-filter kernel (eight waves,
    # one workgroup per CU, 64 or 32 output channels per workgroup)
    (24, 28, 28, 128, 128, (5, 3), (5, 3), "all"),    # 64 channels per workgroup, ragged
    (88, 14, 14, 256, 64, (5, 3), (4, 2), "plain"),   # 32 channels per workgroup
]
# stride 2 (output (H - 1) / 2 + 1): N, H, W, C, K, fx, fw, variant.  The direct kernel
# takes 256 or more input channels; the others check the implicit-GEMM path.
CASES_S2 = [
    (2, 14, 14, 256, 512, (5, 3), (4, 2), "plain"),   # l4.0.c1: four chunks, eight channel tiles
    (3, 7, 7, 256, 64, (6, 3), (4, 1), "all"),        # 4 x 4 outputs per image
    (2, 9, 11, 320, 128, (5, 3), (5, 3), "residual"), # five chunks, odd H and W
    (4, 15, 17, 256, 64, (4, 2), (5, 3), "relu"),     # H != W, ragged last tile
    (1, 1, 1, 256, 64, (5, 3), (5, 3), "affine"),     # one input pixel, one output
    (2, 30, 62, 256, 64, (5, 3), (5, 3), "relu"),     # W + 2 = 64: 11 patch rows, implicit GEMM
    (2, 56, 56, 64, 128, (5, 3), (5, 3), "all"),      # the ResNet18 l2.0.c1 shape, batch 2
    (3, 28, 28, 128, 256, (5, 3), (5, 3), "relu"),    # l3.0.c1
    (2, 13, 9, 64, 64, (5, 3), (5, 3), "residual"),   # odd H, W
]


def post_params(seed, y, K, variant):
    r = np.random.default_rng(seed)
    sd = float(np.std(y)) or 1.0
    a = b = res = None
    if variant in ("affine", "all"):
        a = r.uniform(-0.5, 1.5, K).astype(np.float32)
        b = (r.standard_normal(K) * 0.3 * sd).astype(np.float32)
    if variant in ("residual", "all"):
        res = (r.standard_normal(y.shape) * sd).astype(np.float32)
    relu = variant in ("relu", "all")
    return a, b, res, relu, np.float32(0.4 * sd)


@pytest.mark.parametrize("stride,Nb,H,W,C,K,fx,fw,variant",
                         [(1,) + c for c in CASES] + [(2,) + c for c in CASES_S2])
def test_conv3x3_direct(esb, stride, Nb, H, W, C, K, fx, fw, variant):
    torch = torch_cuda()
    x = wl.random_codes(40 + H + C, (Nb, H, W, C), fx[0])
    w = wl.random_codes(41 + W + K, (K, 3, 3, C), fw[0])
    sd = (stride, stride)
    st, acc_o, y_o = oracle.conv2d(x, w, fx[0], fx[1], ALPHA_X, fw[0], fw[1], ALPHA_W,
                                   stride=sd, pad=(1, 1))
    assert st == 0
    log("conv3x3 direct stride %d %s %s" % (stride, (Nb, H, W, C, K, fx, fw), variant))
    if variant == "plain":
        for want_acc in (True, False):
            acc, y = esb.esb_conv2d(dev(x), fx[0], fx[1], scalar(ALPHA_X), dev(w), fw[0], fw[1],
                                    scalar(ALPHA_W), stride=sd, pad=(1, 1), want_acc=want_acc)
            np.testing.assert_array_equal(host(y).view(np.uint32), y_o.view(np.uint32))
            if want_acc:
                np.testing.assert_array_equal(host(acc), acc_o)
        acc_u, y_u = esb.esb_conv2d(unaligned(torch, x), fx[0], fx[1], scalar(ALPHA_X), dev(w),
                                    fw[0], fw[1], scalar(ALPHA_W), stride=sd, pad=(1, 1))
        np.testing.assert_array_equal(host(acc_u), acc_o)
        np.testing.assert_array_equal(host(y_u).view(np.uint32), y_o.view(np.uint32))
        return
    a, b, res, relu, qa = post_params(7, y_o, K, variant)
    z_o, codes_o = oracle.post(y_o.reshape(-1, K), 5, 3, qa, a=a, bias=b,
                               res=None if res is None else res.reshape(-1, K), relu=relu)
    z_o = z_o.reshape(y_o.shape)
    codes_o = codes_o.reshape(y_o.shape)
    outs = []
    for xin, want_acc in ((dev(x), True), (dev(x), False), (unaligned(torch, x), True)):
        amax = scalar(0.0)
        acc, y, codes = esb.esb_conv2d_post(
            xin, fx[0], fx[1], scalar(ALPHA_X), dev(w), fw[0], fw[1], scalar(ALPHA_W),
            scalar(qa), 5, 3, a=None if a is None else dev(a), b=None if b is None else dev(b),
            residual=None if res is None else dev(res), relu=relu, stride=sd, pad=(1, 1),
            want_codes=True, want_acc=want_acc, want_y=True, absmax=amax)
        np.testing.assert_array_equal(host(y).view(np.uint32), z_o.view(np.uint32))
        np.testing.assert_array_equal(host(codes), codes_o)
        assert host(amax)[0] == np.max(np.abs(z_o))
        if want_acc:
            np.testing.assert_array_equal(host(acc), acc_o)
        outs.append(host(y))
    np.testing.assert_array_equal(outs[0].view(np.uint32), outs[2].view(np.uint32))


def random_shapes(count, seed=2109):
    """Seeded shapes in the direct kernels' domain (channels in multiples of 64, stride 1
    or 2), each at most about 1.5e8 multiply-adds so that the oracle finishes quickly."""
    r = np.random.default_rng(seed)
    out = []
    while len(out) < count:
        st = int(r.choice([1, 2]))
        C = 64 * int(r.choice([1, 2, 3, 4, 5, 8]))
        K = 64 * int(r.choice([1, 2, 3]))
        H, W = int(r.integers(1, 41)), int(r.integers(1, 41))
        Nb = int(r.integers(1, 5))
        P, Q = (H - 1) // st + 1, (W - 1) // st + 1
        if Nb * P * Q * K * 9 * C > 150_000_000:
            continue
        out.append((st, Nb, H, W, C, K))
    return out


@pytest.mark.parametrize("st,Nb,H,W,C,K", random_shapes(24))
def test_conv3x3_direct_random_shapes(esb, st, Nb, H, W, C, K):
    """Plain outputs and int32 sums against the oracle on seeded shapes: ragged tiles, tiles
    across images, odd and even chunk counts, both strides (stride 2 below 256 channels and
    shapes the direct kernels do not take run the implicit GEMM: the same results)."""
    x = wl.random_codes(5000 + H * W + C, (Nb, H, W, C), 5)
    w = wl.random_codes(6000 + K + C, (K, 3, 3, C), 5)
    sd = (st, st)
    status, acc_o, y_o = oracle.conv2d(x, w, 5, 3, ALPHA_X, 5, 3, ALPHA_W, stride=sd, pad=(1, 1))
    assert status == 0
    log("conv3x3 random stride %d %s" % (st, (Nb, H, W, C, K)))
    acc, y = esb.esb_conv2d(dev(x), 5, 3, scalar(ALPHA_X), dev(w), 5, 3, scalar(ALPHA_W),
                            stride=sd, pad=(1, 1), want_acc=True)
    np.testing.assert_array_equal(host(acc), acc_o)
    np.testing.assert_array_equal(host(y).view(np.uint32), y_o.view(np.uint32))


def check_images(esb, Nb, H, W, C, K, form, images, seed):
    """One form of a stride-1 layer on Nb images, the listed ones against the oracle: bit-exact
    sums, outputs and codes, and the maximum of all outputs."""
    x = wl.random_codes(seed, (Nb, H, W, C), 5)
    w = wl.random_codes(seed + 1, (K, 3, 3, C), 5)
    status, acc_o, y_o = oracle.conv2d(np.ascontiguousarray(x[images]), w, 5, 3, ALPHA_X, 5, 3, ALPHA_W,
                                       pad=(1, 1))
    assert status == 0
    log("conv3x3 images %s %s" % ((Nb, H, W, C, K), form))
    head = (dev(x), 5, 3, scalar(ALPHA_X), dev(w), 5, 3, scalar(ALPHA_W))
    if form in ("plain", "sums"):
        acc, y = esb.esb_conv2d(*head, pad=(1, 1), want_acc=form == "sums")
        if form == "sums":
            np.testing.assert_array_equal(host(acc)[images], acc_o)
        np.testing.assert_array_equal(host(y)[images].view(np.uint32), y_o.view(np.uint32))
        return
    a, b, res, _, qa = post_params(13, np.broadcast_to(y_o[:1], (Nb,) + y_o.shape[1:]), K,
                                   {"affine": "affine", "all": "all", "residual": "residual"}.get(form, "none"))
    z_o, codes_o = oracle.post(y_o.reshape(-1, K), 5, 3, qa, a=a, bias=b, relu=True,
                               res=None if res is None else res[images].reshape(-1, K))
    amax = scalar(0.0)
    _, y, codes = esb.esb_conv2d_post(
        *head, scalar(qa), 5, 3, a=None if a is None else dev(a), b=None if b is None else dev(b),
        residual=None if res is None else dev(res), relu=True, pad=(1, 1),
        want_codes=form in ("codes", "y_codes", "all"), want_y=form != "codes", absmax=amax)
    if y is not None:
        np.testing.assert_array_equal(host(y)[images].reshape(-1, K).view(np.uint32), z_o.view(np.uint32))
        assert host(amax)[0] == np.abs(host(y)).max()
    if codes is not None:
        np.testing.assert_array_equal(host(codes)[images].reshape(-1, K), codes_o)


# stride, N, H, W, C, K
HALVED = [
    (1, 1, 7, 7, 384, 64),       # six chunks: three per half; one 64-pixel tile
    (1, 2, 5, 6, 448, 128),      # seven: the second half idles in the last round
    (1, 3, 9, 13, 576, 64),      # nine, ragged last tile
    (2, 2, 14, 14, 512, 128),    # stride 2
    (1, 1, 3, 60, 384, 64),      # wide rows: more patch chunks per thread
    (1, 50, 7, 7, 512, 448),     # 128-pixel tiles, two channel blocks per wave
    (1, 8, 3, 60, 384, 704),     # 128-pixel tiles, wide rows
]


@pytest.mark.parametrize("st,Nb,H,W,C,K", HALVED)
@pytest.mark.parametrize("form", ["plain", "all"])
def test_conv3x3_halved_reduction(esb, st, Nb, H, W, C, K, form):
    """Six or more chunks of input channels with at most one tile per CU: the two halves of a
    workgroup share the chunks and add their sums."""
    x = wl.random_codes(7000 + H + C, (Nb, H, W, C), 5)
    w = wl.random_codes(7100 + W + K, (K, 3, 3, C), 5)
    sd = (st, st)
    status, _, y_o = oracle.conv2d(x, w, 5, 3, ALPHA_X, 5, 3, ALPHA_W, stride=sd, pad=(1, 1))
    assert status == 0
    log("conv3x3 halved stride %d %s %s" % (st, (Nb, H, W, C, K), form))
    head = (dev(x), 5, 3, scalar(ALPHA_X), dev(w), 5, 3, scalar(ALPHA_W))
    if form == "plain":
        _, y = esb.esb_conv2d(*head, stride=sd, pad=(1, 1), want_acc=False)
        np.testing.assert_array_equal(host(y).view(np.uint32), y_o.view(np.uint32))
        return
    a, b, res, relu, qa = post_params(9, y_o, K, "all")
    z_o, codes_o = oracle.post(y_o.reshape(-1, K), 5, 3, qa, a=a, bias=b, res=res.reshape(-1, K),
                               relu=relu)
    amax = scalar(0.0)
    _, y, codes = esb.esb_conv2d_post(*head, scalar(qa), 5, 3, a=dev(a), b=dev(b),
                                      residual=dev(res), relu=relu, stride=sd, pad=(1, 1),
                                      want_codes=True, want_y=True, absmax=amax)
    np.testing.assert_array_equal(host(y).reshape(-1, K).view(np.uint32), z_o.view(np.uint32))
    np.testing.assert_array_equal(host(codes).reshape(-1, K), codes_o)
    assert host(amax)[0] == np.max(np.abs(z_o))


# stride, N, H, W, C, K: one kernel and tile each
OUTPUTS = [
    (1, 1, 11, 13, 64, 64),      # one chunk, 64-pixel tiles, ragged
    (1, 24, 28, 28, 64, 64),     # one chunk, many pixels: codes on the resident-filter kernel
    (1, 24, 28, 28, 128, 64),    # resident filter, 64 channels per workgroup, ragged last tile
    (1, 90, 14, 14, 256, 32 * 6),  # resident filter, 32 channels per workgroup
    (2, 3, 15, 13, 256, 128),    # several chunks, stride 2
    (1, 50, 7, 7, 192, 512),     # several chunks, 128-pixel tiles
    (1, 50, 7, 7, 448, 512),     # halves of the reduction, 128-pixel tiles
    (1, 2, 5, 7, 384, 64),       # halves, 64-pixel tiles
]


@pytest.mark.parametrize("st,Nb,H,W,C,K", OUTPUTS)
@pytest.mark.parametrize("form", ["codes", "relu_y", "in_place", "absmax"])
def test_conv3x3_direct_outputs(esb, st, Nb, H, W, C, K, form):
    """Outputs that leave straight from the accumulators: codes alone, fp32 with ReLU, a
    residual that is the output buffer itself; and the maximum alone, which has none."""
    x = wl.random_codes(8000 + H + C, (Nb, H, W, C), 5)
    w = wl.random_codes(8100 + W + K, (K, 3, 3, C), 5)
    sd = (st, st)
    status, _, y_o = oracle.conv2d(x, w, 5, 3, ALPHA_X, 5, 3, ALPHA_W, stride=sd, pad=(1, 1))
    assert status == 0
    r = np.random.default_rng(11)
    sdev = float(np.std(y_o)) or 1.0
    qa = np.float32(0.4 * sdev)
    res = (r.standard_normal(y_o.shape) * sdev).astype(np.float32) if form == "in_place" else None
    z_o, codes_o = oracle.post(y_o.reshape(-1, K), 5, 3, qa, res=None if res is None else
                               res.reshape(-1, K), relu=form != "in_place")
    log("conv3x3 outputs stride %d %s %s" % (st, (Nb, H, W, C, K), form))
    amax = scalar(0.0)
    y_in = dev(res) if res is not None else None
    _, y, codes = esb.esb_conv2d_post(
        dev(x), 5, 3, scalar(ALPHA_X), dev(w), 5, 3, scalar(ALPHA_W), scalar(qa), 5, 3,
        residual=y_in, y=y_in, relu=form != "in_place", stride=sd, pad=(1, 1),
        want_codes=form == "codes", want_y=form == "relu_y", absmax=amax)
    if form == "codes":
        np.testing.assert_array_equal(host(codes).reshape(-1, K), codes_o)
    elif form != "absmax":
        np.testing.assert_array_equal(host(y).reshape(-1, K).view(np.uint32), z_o.view(np.uint32))
    assert host(amax)[0] == np.max(np.abs(z_o))


# several chunks, 128-pixel tiles, eight, nine and ten patch chunks per thread: N, H, W, C, K
WIDE = [(2, 56, 56, 128, 256), (4, 40, 40, 192, 192), (7, 31, 31, 128, 256), (3, 57, 47, 256, 192)]


@pytest.mark.parametrize("Nb,H,W,C,K", WIDE)
@pytest.mark.parametrize("form", ["plain", "sums", "residual", "codes", "all"])
def test_conv3x3_wide_images(esb, Nb, H, W, C, K, form):
    check_images(esb, Nb, H, W, C, K, form, sorted({0, Nb // 2, Nb - 1}), 9000 + W)


# one chunk: pixels per tile, patch chunks per thread the kernel is built for, H, W, K
ONE_CHUNK = [
    (256, 10, 56, 56, 64),     # the ResNet18 l1 shape: ten patch rows, one per step
    (256, 10, 7, 7, 512),      # tiles over seven images
    (256, 10, 31, 23, 128),    # ragged last tile
    (128, 5, 28, 28, 64),
    (128, 5, 13, 13, 192),     # ragged last tile
    (128, 5, 7, 7, 256),       # tiles over four images
    (128, 10, 56, 56, 64),
    (128, 10, 29, 25, 128),    # ragged last tile
]


@pytest.mark.parametrize("tile,fill,H,W,K", ONE_CHUNK)
@pytest.mark.parametrize("form", ["plain", "sums", "residual", "affine", "codes", "y_codes", "all"])
def test_conv3x3_one_chunk(esb, tile, fill, H, W, K, form):
    """64 input channels on the fewest images whose tiles of 256 or 128 pixels give each CU one:
    more pixels would take the next larger tile (or, for codes, the resident filter)."""
    cus = torch_cuda().cuda.get_device_properties(0).multi_processor_count
    tiles = -(-cus // (K // 64))                   # of each channel tile
    Nb = -(-((tiles - 1) * tile + 1) // (H * W))
    assert -(-Nb * H * W // tile) * (K // 64) >= cus
    assert tile == 256 or -(-Nb * H * W // 256) * (K // 64) < cus
    step = 64 // (W + 2)                           # patch rows that the threads fill at once
    span = (W - 1 + tile - 1) // W                 # output rows of a tile after its first
    rows = span + 2 * ((H - 1 + span) // H) + 3
    assert (5 if tile < 256 and -(-rows // step) <= 5 else 10) == fill
    check_images(esb, Nb, H, W, 64, K, form, sorted({0, Nb // 2, Nb - 1}), 9300 + W + tile)


@pytest.mark.parametrize("st,Nb,H,C,K", [(1, 5400, 56, 256, 64), (2, 45000, 14, 512, 64)])
def test_conv3x3_inputs_past_4_gib(esb, st, Nb, H, C, K):
    """Inputs of more than 2^32 bytes run in parts of whole images: images on both sides of the
    seam, the first and the last against the oracle, the residual and output of each at its place,
    one maximum over all."""
    torch = torch_cuda()
    assert Nb * H * H * C > 2 ** 32
    gen = torch.Generator("cuda").manual_seed(5)
    x = torch.randint(0, 32, (Nb, H, H, C), dtype=torch.uint8, device="cuda", generator=gen)
    w = wl.random_codes(9100, (K, 3, 3, C), 5)
    images = [0, Nb // 2 - 1, Nb // 2, Nb - 1]
    status, _, y_o = oracle.conv2d(host(x[images]), w, 5, 3, ALPHA_X, 5, 3, ALPHA_W, stride=(st, st), pad=(1, 1))
    assert status == 0
    sd = float(np.std(y_o))
    qa = np.float32(0.4 * sd)
    P = y_o.shape[1]
    log("conv3x3 past 4 GiB stride %d %s" % (st, (Nb, H, C, K)))
    head = (x, 5, 3, scalar(ALPHA_X), dev(w), 5, 3, scalar(ALPHA_W))
    y = torch.randn((Nb, P, P, K), device="cuda", generator=gen) * sd     # the residual, replaced
    res = host(y[images])
    z_o, _ = oracle.post(y_o.reshape(-1, K), 5, 3, qa, res=res.reshape(-1, K), relu=True)
    amax = scalar(0.0)
    esb.esb_conv2d_post(*head, scalar(qa), 5, 3, residual=y, y=y, relu=True, stride=(st, st), pad=(1, 1),
                        want_codes=False, absmax=amax)
    np.testing.assert_array_equal(host(y[images]).reshape(-1, K).view(np.uint32), z_o.view(np.uint32))
    assert host(amax)[0] == float(y.abs().max())
    _, codes_o = oracle.post(y_o.reshape(-1, K), 5, 3, qa, relu=True)
    _, _, codes = esb.esb_conv2d_post(*head, scalar(qa), 5, 3, relu=True, stride=(st, st), pad=(1, 1))
    np.testing.assert_array_equal(host(codes[images]).reshape(-1, K), codes_o)
