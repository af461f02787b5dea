"""128 x 128 tiles with columns for some of their eight waves only: the others fetch, and meet the barriers, without multiplying."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
import test_gpu_int8 as I8
import test_gpu_parity as P

pytestmark = pytest.mark.gpu

BF16, F16, F32, E4M3 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32, wl.DTYPE_FP8_E4M3
COLUMNS = [8, 32, 40, 64, 72, 96, 104, 136]        # one wave of four, two, three; the second tile's waves


@pytest.mark.parametrize("force", ["mfma:1", "mfma:2"])
@pytest.mark.parametrize("dtype,out_dtype,trans_b", [(BF16, BF16, 0), (F16, F32, 1)])
@pytest.mark.parametrize("k", [40, 64, 328, 1096])          # one k-tile, ragged and full; fewer and more than the ring holds
def test_matmul(k, dtype, out_dtype, trans_b, force):
    for n in COLUMNS:
        w = wl.Workload(f"mm_cols{n}", "matmul", dtype, out_dtype, C.EPI_BIAS, M=200, N=n, K=k, trans_b=trans_b,
                        dist_b=("normal", 1.0 / np.sqrt(k)), dist_bias=("normal", 0.5))
        P.check_full(w, force=force)


@pytest.mark.parametrize("force", ["mfma:1", "mfma:2"])
@pytest.mark.parametrize("transposed", [0, 1])
@pytest.mark.parametrize("cin", [24, 128])                  # k-tiles that span taps, and that do not
def test_conv(cin, transposed, force):
    for n in COLUMNS:
        w = wl.Workload(f"conv_cols{n}", "conv", BF16, BF16, C.EPI_BIAS_RELU, n=2, H=13, W=11, Cin=cin, Cout=n, KH=4, KW=4, stride=(2, 2), pad=(1, 1),
                        transposed=transposed, dist_b=("normal", float(np.sqrt(2.0 / (16 * cin)))))
        P.check_full(w, force=force)


@pytest.mark.parametrize("force", ["mfma:1", "mfma:2"])
@pytest.mark.parametrize("trans_b", [0, 1])
def test_fp8(trans_b, force):
    for n in (16, 32, 48, 64, 80, 144):
        w = wl.Workload(f"fp8_cols{n}", "matmul", E4M3, BF16, C.EPI_BIAS, M=200, N=n, K=656, trans_b=trans_b,
                        dist_b=("normal", 1.0 / np.sqrt(656)), dist_bias=("normal", 0.5))
        P.check_full(w, force=force)


@pytest.mark.parametrize("cfg", [1, 2])
def test_int8(cfg):
    for n in (16, 32, 48, 64, 80, 144):
        I8.test_matmul_int8_row_major_b_on_mfma(cfg, (200, n, 656))
        I8.test_matmul_int8_kmajor(cfg, (200, n, 656))
        I8.test_matmul_int8_unfolded_batch_norm_is_bit_exact(f"mfma:{cfg}", True, (200, n, 656))
        I8.test_matmul_int8_unfolded_batch_norm_is_bit_exact(f"mfma:{cfg}", False, (200, n, 656))
