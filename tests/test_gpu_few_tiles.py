"""Matrix-unit kernels for problems with few tiles, against the oracle."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
from test_gpu_bstat import run_case

pytestmark = pytest.mark.gpu

BF16, F16, F32, E4M3 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32, wl.DTYPE_FP8_E4M3
# one rounding to the output type; fp32 output: sums of K products in another order
TOL = {BF16: T.TIGHT[BF16], F16: T.TIGHT[F16], F32: T.TIGHT[F32]}


@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("M,N,K,tile", [(2100, 2049, 37, "128x128"), (2048, 2048, 37, "64x128"), (65, 131, 301, "64x128")])
def test_gather_tiles(M, N, K, tile, trans_b):
    """Either side of the line between the two row tiles of the gathering kernel."""
    err, kern = run_case(1, M, N, K, BF16, BF16, trans_b, C.EPI_BIAS, pad_ld=1, force="gather")
    assert tile in kern, kern
    assert err <= TOL[BF16], err
