"""The tiles of the gathering matrix-unit kernel (128 and 64 rows, 128 rows in the deep form) on every mode that it is built for: the cases of
the automatic choice, which takes one of the two by size, and contractions from one k-tile of 32 over the last one that only has
careful steps (five) into the unrolled steady state."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
import test_gpu_gather as G
from test_gpu_bstat import run_case

pytestmark = pytest.mark.gpu

BF16, F16, F32 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32
NAMES = {"gather:0": "gather_128x128x32", "gather:1": "gather_64x128", "gather:4": "gather_128x128x64", "gather:5": "gather_128x128x64"}
rows = pytest.mark.parametrize("force", list(NAMES))


@rows
@pytest.mark.parametrize("dtype,out_dtype", [(BF16, BF16), (F16, F16), (BF16, F32), (F16, F32)])
@pytest.mark.parametrize("trans_b", [0, 1])
def test_matmul(force, dtype, out_dtype, trans_b):
    nan = 0x7FC0 if dtype == BF16 else 0x7E00
    for M, N, K, pad in [(300, 261, 1143, 3), (129, 127, 37, 1), (65, 131, 301, 1), (63, 129, 160, 1), (191, 260, 193, 5), (257, 384, 4097, 1)]:
        lda, ldb = K + pad, (K if trans_b else N) + 1
        a = wl.tensor((M, lda), dtype, 1, "normal")
        b = wl.tensor(((N if trans_b else K), ldb), dtype, 2, "normal", 1.0 / np.sqrt(K))
        a[:, K:] = nan
        b[:, ldb - 1:] = nan
        bias = wl.tensor((N,), F32, 3, "normal", 0.5)
        err, kern = G.run_views(a, b, bias, M, N, K, lda, ldb, N, dtype, out_dtype, trans_b, C.EPI_BIAS_GELU_TANH, alpha=0.75, force=force)
        assert NAMES[force] in kern, kern
        assert err <= T.TIGHT[out_dtype], (M, N, K, err)


@rows
@pytest.mark.parametrize("a_off,b_off", [(1, 0), (0, 3), (5, 7)])
def test_unaligned_bases(force, a_off, b_off):
    M, N, K = 200, 264, 328
    a = wl.tensor((M * K + 16,), BF16, 1, "normal")
    b = wl.tensor((K * N + 16,), BF16, 2, "normal", 1.0 / np.sqrt(K))
    err, kern = G.run_views(a, b, None, M, N, K, K, N, N, BF16, BF16, 0, C.EPI_RELU, force=force, a_off=a_off, b_off=b_off)
    assert NAMES[force] in kern and err <= T.TIGHT[BF16], (kern, err)


@rows
@pytest.mark.parametrize("dtype,out_dtype", [(F16, F32), (BF16, BF16)])
@pytest.mark.parametrize("case", [
    # n, H, W, Cin, Cout, KH, KW, stride, pad, dil
    (2, 44, 44, 127, 24, 3, 3, (2, 2), (0, 0), (1, 1)),
    (1, 20, 19, 127, 136, 3, 3, (1, 1), (1, 1), (1, 1)),
    (2, 15, 17, 9, 40, 5, 3, (1, 2), (2, 1), (2, 1)),
    (1, 30, 30, 3, 64, 7, 7, (2, 2), (3, 3), (1, 1)),
    (1, 12, 13, 20, 40, 3, 3, (1, 1), (1, 1), (1, 1)),
    (1, 12, 12, 30, 261, 1, 1, (1, 1), (0, 0), (1, 1)),
    (6, 9, 11, 8, 12, 2, 2, (1, 1), (0, 1), (1, 1)),
])
def test_conv(case, dtype, out_dtype, force):
    n, H, W, Cin, Cout, KH, KW, stride, pad, dil = case
    w = wl.Workload("conv_gather_rows", "conv", dtype, out_dtype, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout, KH=KH, KW=KW,
                    stride=stride, pad=pad, dil=dil, dist_b=("normal", float(np.sqrt(2.0 / (KH * KW * Cin)))))
    with T.forced_kernel(force):
        G.check_workload(w, NAMES[force])


@rows
@pytest.mark.parametrize("K", [61, 333])
def test_batched(force, K):
    w = wl.Workload("bmm_gather_rows", "batched", BF16, F32, C.EPI_NONE, alpha=0.5, batch=3, M=131, N=77, K=K, dist_b=("normal", K ** -0.5))
    with T.forced_kernel(force):
        G.check_workload(w, NAMES[force])


@pytest.mark.parametrize("M,N,K,kernel", [
    (1025, 1921, 513, "128x128x64"), (1025, 1921, 511, "64x128x32"), (1024, 2047, 513, "64x128x64"),       # 272 tiles of 64 rows, 256
    (2048, 2047, 601, "128x128x64"), (2049, 2047, 601, "128x128x32"),                                      # 256 tiles of 128 rows, 272
])
def test_dispatch(M, N, K, kernel):
    err, kern = run_case(1, M, N, K, BF16, BF16, 0, C.EPI_NONE, pad_ld=1, force=None, bias_on=False)
    assert kernel in kern and err <= T.TIGHT[BF16], (kern, err)


@pytest.mark.parametrize("hw,cout,kernel", [(65, 512, "128x128x64"), (91, 512, "64x128x32"), (110, 512, "64x128x32"), (112, 512, "128x128x32")])
def test_dispatch_conv(hw, cout, kernel):
    """4225 rows x 4 columns of tiles: 268 of 64 rows; 8281: 260 of 128 rows; 12100: 760 of 64 rows; 12544: 784."""
    w = wl.Workload("gather_form", "conv", BF16, BF16, C.EPI_BIAS_RELU, n=1, H=hw + 1, W=hw + 1, Cin=9, Cout=cout, KH=2, KW=2, dist_b=("normal", 0.2))
    G.check_workload(w, kernel)


@pytest.mark.parametrize("cin,cout,kernel", [(127, 32, "128x128x32"), (127, 40, "64x128x32"), (100, 32, "64x128x32")])
def test_dispatch_conv_narrow(cin, cout, kernel):
    """600 tiles of 64 rows, 7 x 7: up to 32 columns, with channels that a row of taps does not shorten, on 128 rows."""
    w = wl.Workload("gather_narrow", "conv", BF16, BF16, C.EPI_BIAS_RELU, n=1, H=196, W=196, Cin=cin, Cout=cout, KH=7, KW=7, pad=(3, 3),
                    dist_b=("normal", float(np.sqrt(2.0 / (49 * cin)))))
    G.check_workload(w, kernel)
