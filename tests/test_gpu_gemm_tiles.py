"""Dense products on both sides of the rules that choose tile and split, vs the oracle: 64 x 64 tiles
up to two (three for K <= 1024) per compute unit, 128 x 128 beyond, and the reduction split or
whole by K and the fill of the tiles.  Int32 sums bit for bit, fp32 outputs equal; a workspace of
exactly the size the library asks for, its bytes past that untouched."""
import numpy as np
import pytest

import oracle
from gpuutil import dev, host, log, torch_cuda, scalar
from paper_2109_03513_amd import workloads as wl

pytestmark = pytest.mark.gpu


def check(M, N, K, f, ws, seed):
    from paper_2109_03513_amd import esb
    torch = torch_cuda()
    A = wl.random_codes(seed, (M, K), 8)
    B = wl.random_codes(seed + 1, (N, K), 8)
    need = esb.esb_gemm_workspace_size(M, N, K, *f, *f) if ws else 0
    work = torch.full((need + 64,), 0xA5, dtype=torch.uint8, device="cuda") if ws else None
    log("gemm tiles %s ws %d" % ((M, N, K, f), need))
    acc, y = esb.esb_gemm(dev(A), *f, scalar(0.37), dev(B), *f, scalar(0.021),
                          workspace=None if work is None else work[:need] if need else None)
    rows, cols = (np.array([i for i in sorted({0, 63, 64, 127, 128, n // 2, n - 1}) if i < n])
                  for n in (M, N))
    s, oacc, oy = oracle.gemm(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[cols]), *f, 0.37,
                              *f, 0.021)
    assert s == 0
    np.testing.assert_array_equal(host(acc)[np.ix_(rows, cols)], oacc)
    np.testing.assert_array_equal(host(y)[np.ix_(rows, cols)], oy)
    assert (host(y) == (host(acc) * np.float32(np.float32(0.37) * np.float32(0.021)) *
                        np.float32(2.0 ** (-2 * (f[1] - 1)))).astype(np.float32)).all()
    if work is not None:
        assert (host(work)[need:] == 0xA5).all()


def side(tiles, k):
    """Rows of a product k tiles of 64 wide with about that many tiles of 64 x 64 in all."""
    return 64 * (tiles // k) - 1


@pytest.mark.parametrize("per,K", [(2, 1040), (3, 1024), (3, 1040)])
@pytest.mark.parametrize("f", [(5, 3), (3, 2)])
@pytest.mark.parametrize("over", [False, True])
def test_tiles_per_cu(per, K, f, over):
    cus = torch_cuda().cuda.get_device_properties(0).multi_processor_count
    check(side(per * cus, 16) + (64 if over else 0), 1021, K, f, False, 500 + per)


@pytest.mark.parametrize("M,N,K", [
    (1000, 1000, 4096), (1000, 1000, 4112), (65, 8192, 3584), (65, 8192, 3600),    # four ranges, 64 tiles
    (768, 1400, 6000), (768, 1400, 6016), (1200, 1200, 8192), (1200, 1200, 8208),  # four, three ranges
    (500, 1000, 4080), (500, 1000, 4096)])                                        # 128 tiles of 64 x 64
@pytest.mark.parametrize("f", [(4, 2), (3, 2)])
def test_split_limits(M, N, K, f):
    check(M, N, K, f, True, 520)
