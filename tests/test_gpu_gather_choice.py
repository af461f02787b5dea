"""Where the gathering kernel takes products with few outputs from the generic one: either side of each line of the rule."""
import pytest

import workloads as wl
from workloads import configs as C
from test_gpu_bstat import run_case
from test_gpu_few_tiles import TOL

pytestmark = pytest.mark.gpu

BF16 = wl.DTYPE_BF16


@pytest.mark.parametrize("batch,M,N,K,trans_b,gather", [
    (1, 64, 65, 17, 0, True), (1, 63, 65, 17, 0, False), (1, 63, 65, 65, 0, True), (1, 63, 65, 63, 0, False), (1, 200, 15, 65, 0, False), (1, 1, 17, 65, 0, True),
    (512, 17, 17, 65, 0, True), (513, 17, 17, 65, 0, False), (513, 17, 17, 97, 0, True), (2049, 5, 17, 97, 0, False), (2049, 5, 17, 129, 0, True),
    (300, 1, 129, 65, 0, True), (300, 1, 129, 65, 1, False), (256, 1, 129, 65, 1, True), (513, 1, 70, 65, 1, True), (171, 3, 513, 65, 1, True),
])
def test_dispatch(batch, M, N, K, trans_b, gather):
    err, kern = run_case(batch, M, N, K, BF16, BF16, trans_b, C.EPI_NONE, pad_ld=1, force=None, bias_on=False)
    assert ("gather" in kern) == gather and ("generic" in kern) != gather, kern
    assert err <= TOL[BF16], err
