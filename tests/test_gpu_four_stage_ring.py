"""The 128 x 128 tile with a four-stage ring (tile configuration 2) on every mode and type that it is built for: the cases of the
other configurations, and sweeps over the number of k-tiles (three are in flight: fewer than that, exactly that, and
the steady state that refills the ring)."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
import test_gpu_conv_variants as V
import test_gpu_int8 as I8
import test_gpu_parity as P
import test_gpu_residual as R

pytestmark = pytest.mark.gpu

BF16, F16, F32 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32
KS = [8, 40, 64, 72, 128, 136, 192, 200, 256, 264, 328, 392, 1096]


@pytest.fixture(autouse=True)
def ran_on_the_ring():
    """Every case below forces the configuration; the name of the last kernel shows that it ran."""
    import paper_2603_06731_amd as pbk
    yield
    assert "128x128x64_w2x4_s4" in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()


@pytest.mark.parametrize("dtype,out_dtype", [(BF16, BF16), (F16, F32)])
@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("k", KS)
def test_matmul_k_sweep(k, trans_b, dtype, out_dtype):
    w = wl.Workload(f"mm_ring_k{k}", "matmul", dtype, out_dtype, C.EPI_BIAS, M=300, N=264, K=k, trans_b=trans_b,
                    dist_b=("normal", 1.0 / np.sqrt(k)), dist_bias=("normal", 0.5))
    P.check_full(w, force="mfma:2")


def test_batched():
    w = wl.Workload("bmm_ring", "batched", BF16, F32, C.EPI_NONE, alpha=0.5, batch=3, M=264, N=256, K=392, dist_b=("normal", 0.05))
    P.check_full(w, force="mfma:2")


@pytest.mark.parametrize("case", P.CONV_SMALL + [(1, 13, 12, 96, 136, 3, 3, (1, 1), (1, 1), (1, 1))])
@pytest.mark.parametrize("dtype", [BF16, F16])
def test_conv(case, dtype):
    n, H, W, Cin, Cout, KH, KW, stride, pad, dil = case
    w = wl.Workload("conv_ring", "conv", dtype, dtype, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout, KH=KH, KW=KW,
                    stride=stride, pad=pad, dil=dil, dist_b=("normal", float(np.sqrt(2.0 / (KH * KW * Cin)))))
    P.check_full(w, force="mfma:2")


@pytest.mark.parametrize("case", V.PAD4)
def test_conv_pad4(case):
    V.test_conv_pad4(case, 2)


@pytest.mark.parametrize("case", V.CONVT)
def test_conv_transpose(case):
    V.test_conv_transpose(case, 2)


@pytest.mark.parametrize("dtype", P.FP8_TYPES)
@pytest.mark.parametrize("out_dtype", [BF16, F16, F32])
@pytest.mark.parametrize("k", [16, 80, 128, 208, 400, 1040, 2192])
def test_fp8_k_major(dtype, out_dtype, k):
    w = wl.Workload(f"fp8_ring_k{k}", "matmul", dtype, out_dtype, C.EPI_BIAS_GELU_TANH, alpha=0.5, M=300, N=261, K=k, trans_b=1,
                    dist_b=("normal", 1.0 / np.sqrt(k)), dist_bias=("normal", 0.5))
    P.check_full(w, force="mfma:2")


@pytest.mark.parametrize("dtype", P.FP8_TYPES)
@pytest.mark.parametrize("mnk", [(300, 272, 208), (256, 512, 128), (33, 144, 4096)])
def test_fp8_row_major(dtype, mnk):
    P.test_fp8_matmul_row_major_b_on_mfma(dtype, 2, mnk)


@pytest.mark.parametrize("dtype", P.FP8_TYPES)
@pytest.mark.parametrize("case", [(2, 14, 13, 32, 48, 3, 3, (1, 1), (1, 1), (1, 1)), (1, 17, 16, 128, 64, 3, 3, (2, 2), (1, 1), (1, 1)),
                                  (2, 12, 12, 48, 80, 2, 3, (1, 2), (0, 2), (2, 1))])
def test_fp8_conv(dtype, case):
    P.test_fp8_conv_on_mfma(dtype, 2, case)


@pytest.mark.parametrize("mnk", I8.SHAPES)
def test_int8_k_major(mnk):
    I8.test_matmul_int8_kmajor(2, mnk)


@pytest.mark.parametrize("mnk", [(300, 272, 208), (256, 512, 128), (33, 144, 4096)])
def test_int8_row_major(mnk):
    I8.test_matmul_int8_row_major_b_on_mfma(2, mnk)


@pytest.mark.parametrize("geom", [((1, 1), (1, 1), (1, 1)), ((2, 2), (1, 1), (1, 1)), ((1, 2), (2, 0), (2, 1))])
def test_int8_conv(geom):
    I8.test_conv_int8_on_mfma(2, geom)


@pytest.mark.parametrize("out_int8", [True, False])
@pytest.mark.parametrize("mnk", [(300, 264, 208), (130, 272, 4096)])
def test_int8_batch_norm(out_int8, mnk):
    I8.test_matmul_int8_unfolded_batch_norm_is_bit_exact("mfma:2", out_int8, mnk)


@pytest.mark.parametrize("mnk", [(300, 264, 200), (256, 512, 64), (33, 520, 136), (130, 264, 1096)])
@pytest.mark.parametrize("dtype,out_dtype", [(BF16, BF16), (F16, F32)])
def test_residual(mnk, dtype, out_dtype):
    R.test_matmul_residual(2, mnk, dtype, out_dtype)


@pytest.mark.parametrize("dtype,out_dtype", [(BF16, BF16), (F16, F32)])
@pytest.mark.parametrize("n,ldc,ldr", [(257, 257, 257), (264, 267, 269)])
def test_residual_direct_stores(dtype, out_dtype, n, ldc, ldr):
    R.test_matmul_residual_direct_stores_on_mfma(2, dtype, out_dtype, n, ldc, ldr)


def test_conv_residual():
    R.test_conv_residual_block(2)
