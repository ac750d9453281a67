"""The general contraction's loaders vs the oracle, bit for bit: rows of any length and
alignment (16-byte loads at any address, their tails at every remainder), rows too short for
them, the KN layout in 4 x 4 blocks, row pitches and base addresses of their own, formats in one
and in two int8 planes.  Nothing outside the output is written."""
import ctypes

import numpy as np
import pytest

import oracle
from gpuutil import dev, host, log, scalar
from paper_2109_03513_amd import workloads as wl

pytestmark = pytest.mark.gpu


def run(M, N, K, fa, fb, layout, padA, padB, offA, offB, seed):
    from paper_2109_03513_amd import esb
    torch = pytest.importorskip("torch")
    rows, cols = (N, K) if layout == 0 else (K, N)
    A = wl.random_codes(seed, (M, K + padA), 8)
    B = wl.random_codes(seed + 1, (rows, cols + padB), 8)
    st, oacc, oy = oracle.gemm(np.ascontiguousarray(A[:, :K]), np.ascontiguousarray(B[:, :cols]),
                               *fa, 0.37, *fb, 0.021, b_layout=layout)
    assert st == 0
    # the last code of each operand is the last byte of its buffer
    bufs = []
    for a, off, pad in ((A, offA, padA), (B, offB, padB)):
        t = torch.zeros(off + a.size - pad, dtype=torch.uint8, device="cuda")
        t[off:].copy_(dev(a).reshape(-1)[:a.size - pad])
        bufs.append(t[off:])
    ldc = N + 3
    acc = torch.full((M, ldc), -7, dtype=torch.int32, device="cuda")
    y = torch.full((M, ldc), -7.0, dtype=torch.float32, device="cuda")
    a, b = scalar(0.37), scalar(0.021)
    esb._check("esb_gemm", esb.lib().esb_gemm(
        M, N, K, ctypes.c_void_p(bufs[0].data_ptr()), K + padA, *fa, esb._ptr(a),
        ctypes.c_void_p(bufs[1].data_ptr()), cols + padB, *fb, esb._ptr(b), layout, esb._ptr(acc),
        esb._ptr(y), ldc, esb._stream(None)))
    np.testing.assert_array_equal(host(acc)[:, :N], oacc)
    np.testing.assert_array_equal(host(y)[:, :N], oy)
    assert (host(acc)[:, N:] == -7).all() and (host(y)[:, N:] == -7.0).all()


@pytest.mark.parametrize("K", [1, 7, 15, 16, 17, 23, 24, 25, 31, 33, 47, 63, 64, 65, 127, 333])
@pytest.mark.parametrize("fa,fb", [((5, 3), (5, 3)), ((6, 3), (6, 3)), ((3, 2), (8, 5))])
def test_rows_of_any_length(K, fa, fb):
    log("gemm K=%d %s %s" % (K, fa, fb))
    run(33, 21, K, fa, fb, 0, 0, 0, 1, 3, 300 + K)


@pytest.mark.parametrize("M,N,K,layout,padA,padB,offA,offB", [
    (70, 130, 100, 0, 5, 0, 2, 7), (300, 200, 129, 0, 0, 11, 5, 0), (1, 1, 18, 0, 1, 1, 0, 9),
    (9, 1, 40, 1, 0, 0, 3, 1), (65, 3, 77, 1, 2, 1, 0, 5), (130, 4, 64, 1, 0, 4, 0, 0),
    (40, 5, 3, 1, 0, 0, 1, 2), (257, 131, 65, 1, 3, 2, 1, 3), (600, 520, 50, 1, 0, 0, 0, 1),
    (2300, 2100, 37, 0, 0, 0, 1, 1)])     # 128 x 128 tiles
@pytest.mark.parametrize("fa,fb", [((5, 3), (4, 2)), ((7, 4), (5, 3)), ((5, 3), (8, 5))])
def test_layouts_and_pitches(M, N, K, layout, padA, padB, offA, offB, fa, fb):
    log("gemm %s %s %s" % ((M, N, K, layout, padA, padB, offA, offB), fa, fb))
    run(M, N, K, fa, fb, layout, padA, padB, offA, offB, 400 + M)
