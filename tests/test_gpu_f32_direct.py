"""The fp32 kernel that loads its operands straight into registers: k split over waves, 32 x 32 tiles, and its place in the dispatcher."""
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
from test_gpu_small_f32 import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("M,N,K,lds,kernel", [
    (16, 16, 4096, (None, None, None), "small_f32_16x16"),           # sixteen waves
    (33, 130, 1037, (None, None, None), "small_f32_16x16"),          # waves with unequal shares, the last one ragged
    (520, 512, 250, (None, None, None), "small_f32_16x16"),   # beyond one tile per SIMD
    (768, 783, 67, (None, None, None), "small_f32_16x16"),    # 2352 tiles: odd N, no pairs of columns
    (785, 786, 131, (None, None, None), "small_f32_32x32"),   # 2500: N even, rows of B only 8-byte aligned, last pair at the edge
    (800, 770, 64, (None, 786, 772), "small_f32_32x32"),      # one full register set, padded rows
    (801, 801, 65, (68, 804, 803), "small_f32_32x32"),        # everything odd
    (1024, 1024, 128, (None, None, None), "small_f32_32x32"),
    (1025, 1024, 32, (None, None, None), "mfma_f32"),          # 4160 tiles
    (1024, 1024, 32, (None, None, None), "mfma_f32"),          # 4096, a short contraction
    (1, 36864, 16, (None, None, None), "small_f32_16x16"), (1, 36865, 16, (None, None, None), "generic"),     # 2304 and 2305 tiles, mostly empty
    (3, 38401, 32, (None, None, None), "generic"), (3, 38401, 33, (None, None, None), "small_f32_16x16"),
    (4, 38401, 20, (None, None, None), "small_f32_16x16"), (38401, 5, 20, (None, None, None), "small_f32_16x16"),   # 2401, half of a 32 x 32 tile empty
    (16, 56000, 512, (None, None, None), "small_f32_16x16"),   # 3500
    (33, 15000, 48, (None, None, None), "small_f32_32x32"),    # 938 tiles of 32 x 32
    (33, 20000, 41, (None, None, None), "small_f32_16x16"), (33, 20000, 40, (None, None, None), "generic"),   # 1250: more than waves at once
    (801, 803, 33, (None, None, None), "small_f32_32x32"), (801, 803, 30, (None, None, None), "generic"),     # rows of C not aligned
    (60, 16001, 32, (None, None, None), "generic"),
])
def test_parity_and_dispatch(M, N, K, lds, kernel, trans_b):
    lda, ldb, ldc = lds
    if trans_b:
        ldb = None if ldb is None else K + 5
    err, kern = run(M, N, K, trans_b, C.EPI_BIAS_RELU, lda=lda, ldb=ldb, ldc=ldc, alpha=0.75)
    assert kernel in kern, kern
    assert err <= T.TOL_F32, err


@pytest.mark.parametrize("batch,M,N,K,trans_b,kernel", [
    (1000, 3, 50, 16, 0, "generic"), (1000, 3, 50, 33, 0, "small_f32_16x16"), (1000, 3, 50, 512, 0, "small_f32_32x32"),
    (1000, 3, 50, 512, 1, "small_f32_16x16"), (2000, 2, 30, 16, 0, "small_f32_16x16"), (1000, 30, 30, 16, 0, "small_f32_32x32"),
    (450, 33, 46, 64, 0, "small_f32_16x16"), (450, 33, 46, 65, 0, "generic"), (450, 33, 46, 65, 1, "small_f32_16x16"), (450, 33, 46, 63, 1, "generic"),
])
def test_dispatch_of_batches(batch, M, N, K, trans_b, kernel):
    err, kern = run(M, N, K, trans_b, C.EPI_NONE, batch=batch)
    assert kernel in kern and err <= T.TOL_F32, (kern, err)


def test_residual_and_batch():
    err, kern = run(790, 780, 40, 0, C.EPI_GELU_TANH, residual=True)
    assert "small_f32_32x32" in kern and err <= T.TOL_F32, (kern, err)
    err, kern = run(100, 900, 150, 0, C.EPI_BIAS, batch=8)
    assert "small_f32_32x32" in kern and err <= T.TOL_F32, (kern, err)


def test_repeats():
    """The waves' sums are added in a fixed order: the same bits call after call."""
    import torch
    import paper_2603_06731_amd as pbk
    M, N, K = 70, 90, 2050
    a, b = torch.randn(M, K, device="cuda"), torch.randn(K, N, device="cuda")
    out, first = torch.empty(M, N, device="cuda"), None
    for _ in range(8):
        out.fill_(float("nan"))
        assert pbk.pbk_matmul(a, b, out, None, M, N, K, K, N, N, wl.DTYPE_F32, wl.DTYPE_F32, 0, 1.0, 0) == 0
        first = out.clone() if first is None else first
        assert torch.equal(out, first)
    ref = a.double() @ b.double()
    # fp32 sums of K terms of order one: well below K^(1/2) * 2^-24 * K^(1/2)
    assert float((first.double() - ref).abs().max()) <= K * 2.0 ** -24 * 4
