"""128 x 128 tiles on four waves (16-bit plain products of one or two k-tiles that load nothing in the epilogue): parity with the oracle at the
edges of tiles and k-tiles, and either side of each line of the rule that chooses them."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
import test_gpu_parity as P
from test_gpu_bstat import run_case
from test_gpu_few_tiles import TOL

pytestmark = pytest.mark.gpu

BF16, F16, F32 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32


@pytest.mark.parametrize("dtype,out_dtype,epi", [(BF16, BF16, C.EPI_NONE), (F16, F16, C.EPI_RELU), (BF16, F32, C.EPI_BIAS_GELU_TANH)])
@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("k", [8, 64, 72, 96, 128, 200])
def test_parity(k, trans_b, dtype, out_dtype, epi):
    import paper_2603_06731_amd as pbk
    w = wl.Workload(f"four_waves_k{k}", "batched", dtype, out_dtype, epi, batch=2, M=129, N=264, K=k, trans_b=trans_b,
                    dist_b=("normal", 1.0 / np.sqrt(k)), dist_bias=("normal", 0.5))
    P.check_full(w, force="mfma:3")
    assert "128x128x64_w2x2_s2" in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()


@pytest.mark.parametrize("batch,M,N,K,out_dtype,epi,four", [
    (33, 264, 320, 160, BF16, C.EPI_NONE, True), (33, 264, 320, 168, BF16, C.EPI_NONE, False),
    (37, 264, 320, 96, BF16, C.EPI_NONE, True), (37, 264, 320, 104, BF16, C.EPI_NONE, False), (33, 264, 320, 32, F32, C.EPI_NONE, False),
    (33, 264, 320, 32, BF16, C.EPI_BIAS, False), (33, 264, 320, 32, BF16, C.EPI_RELU, True), (16, 384, 640, 64, BF16, C.EPI_NONE, False),
    (129, 100, 248, 64, BF16, C.EPI_NONE, False), (112, 130, 256, 64, BF16, C.EPI_NONE, True), (113, 130, 256, 64, BF16, C.EPI_NONE, False),
])
def test_dispatch(batch, M, N, K, out_dtype, epi, four):
    """297 tiles; 333; 240; 258 with few columns, 448, 452."""
    err, kern = run_case(batch, M, N, K, BF16, out_dtype, 0, epi, force=None, bias_on=epi == C.EPI_BIAS)
    assert ("128x128x64_w2x2_s2" in kern) == four, kern
    assert err <= TOL[out_dtype], err


@pytest.mark.parametrize("dtype,kernel", [("bf16", "128x128x64_w2x2"), ("e4m3", "generic")])
def test_more_entries_than_a_launch_holds(dtype, kernel):
    """2^23 entries of one row, each with a tile of its own, which has 512 threads on eight waves: a launch holds fewer than 2^32 threads.  B is shared
    (stride 0)."""
    import torch
    import paper_2603_06731_amd as pbk
    n, k = 2 ** 23, 16
    g = torch.Generator(device="cuda").manual_seed(3)
    td, code, raw = (torch.bfloat16, pbk.PBK_BF16, lambda x: x) if dtype == "bf16" else (torch.float8_e4m3fn, pbk.PBK_FP8_E4M3, lambda x: x.view(torch.uint8))
    A, B = (torch.randn(r, k, generator=g, device="cuda").to(td) for r in (n, k))
    out = torch.full((n, k), float("nan"), dtype=torch.bfloat16, device="cuda")
    with T.forced_kernel(None):
        st = pbk.pbk_batched_matmul(raw(A), raw(B), out, None, n, 1, k, k, k, k, k, k, 0, k, code, pbk.PBK_BF16, 0, 1.0, 0)
    assert st == 0 and kernel in pbk.pbk_last_kernel(), (st, pbk.pbk_last_kernel())
    for i in range(0, n, 2 ** 20):
        ref = A[i:i + 2 ** 20].float() @ B.float()
        # one rounding to bf16 (2^-9 of the value), fp32 sums of sixteen terms of order one
        assert bool(((out[i:i + 2 ** 20].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5).all())
