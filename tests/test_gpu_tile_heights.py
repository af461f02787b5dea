"""The pair pipeline on tiles of 224 to 128 rows and 256 columns (mfma:10 to 13) and of 256 to 448 rows and 128 columns (mfma:14 to 17): every number of k-tiles that its prologue, steady state and
drain tell apart, both layouts of B, convolutions, 8-bit types, and rows either side of a tile's edge; against the oracle."""
import numpy as np
import pytest

import workloads as wl
import pbk_testlib as T
from workloads import configs as C
from test_gpu_parity import check_full
from test_gpu_int8 import params, run_matmul

pytestmark = pytest.mark.gpu

F32, BF16, F16, E4M3, E5M2 = wl.DTYPE_F32, wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_FP8_E4M3, wl.DTYPE_FP8_E5M2
HEIGHT = {10: 224, 11: 192, 12: 160, 13: 128}
NARROW = {14: 256, 15: 320, 16: 384, 17: 448}            # convolutions
CFGS = sorted(HEIGHT)


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("k", [8, 64, 72, 128, 160, 200, 232, 264, 328, 1096])
def test_k_tiles(cfg, trans_b, k):
    w = wl.Workload(f"height_k{k}", "matmul", BF16, BF16, C.EPI_BIAS, M=HEIGHT[cfg] + 76, N=520, K=k, trans_b=trans_b,
                    dist_b=("normal", 1.0 / np.sqrt(k)), dist_bias=("normal", 0.5))
    check_full(w, force=f"mfma:{cfg}", expect_kernel=f"{HEIGHT[cfg]}x256x32")


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("rows", [-1, 0, 1, "half"])
@pytest.mark.parametrize("out_dtype", ["same", "f32"])
def test_rows(cfg, rows, out_dtype):
    h = HEIGHT[cfg]
    m = h // 2 + 1 if rows == "half" else 2 * h + rows
    w = wl.Workload(f"height_m{m}", "batched", F16, F16 if out_dtype == "same" else F32, C.EPI_NONE, alpha=0.5, batch=2, M=m, N=264, K=392,
                    dist_b=("normal", 0.05))
    check_full(w, force=f"mfma:{cfg}", expect_kernel=f"{h}x256x32")


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("case", [(3, 9, 9, 64, 8, 1, 1), (2, 14, 13, 64, 264, 3, 1), (1, 23, 21, 128, 136, 3, 2), (2, 17, 19, 192, 72, 2, 1)])
def test_conv(cfg, case):
    n, H, W, Cin, Cout, k, s = case
    w = wl.Workload("height_conv", "conv", BF16, BF16, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout, KH=k, KW=k, stride=(s, s),
                    pad=(k // 2, k // 2), dist_b=("normal", float(np.sqrt(2.0 / (k * k * Cin)))))
    check_full(w, force=f"mfma:{cfg}", expect_kernel=f"{HEIGHT[cfg]}x256x32")


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("dtype,k", [(E4M3, 16), (E4M3, 144), (E4M3, 512), (E5M2, 656), (E4M3, 1296)])
def test_fp8(cfg, dtype, k):
    w = wl.Workload(f"height_fp8_k{k}", "matmul", dtype, BF16, C.EPI_BIAS, M=HEIGHT[cfg] + 44, N=517, K=k, trans_b=1,
                    dist_b=("normal", 1.0 / np.sqrt(k)), dist_bias=("normal", 0.5))
    check_full(w, force=f"mfma:{cfg}", expect_kernel=f"{HEIGHT[cfg]}x256x32")


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("k", [16, 144, 400, 1296])
def test_int8(cfg, k):
    import oracle
    m, n = HEIGHT[cfg] + 44, 528
    A, B, q = wl.int8_tensor((m, k), 1), wl.int8_tensor((n, k), 2), params(n, 3)
    got, kernel = run_matmul(A, B, q, 1, True, f"mfma:{cfg}")
    assert f"{HEIGHT[cfg]}x256x32" in kernel, kernel
    assert np.array_equal(got, oracle.matmul_int8(A, B, trans_b=1, **q))


@pytest.mark.parametrize("cfg", sorted(NARROW))
@pytest.mark.parametrize("case", [(3, 9, 9, 64, 8, 1, 2), (2, 21, 21, 64, 128, 3, 1), (1, 43, 21, 128, 136, 3, 2), (2, 17, 31, 192, 72, 2, 1)])
def test_conv_narrow(cfg, case):
    n, H, W, Cin, Cout, k, s = case
    w = wl.Workload("narrow_conv", "conv", F16, F16, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout, KH=k, KW=k, stride=(s, s),
                    pad=(k // 2, k // 2), dist_b=("normal", float(np.sqrt(2.0 / (k * k * Cin)))))
    check_full(w, force=f"mfma:{cfg}", expect_kernel=f"{NARROW[cfg]}x128x32")


@pytest.mark.parametrize("cfg", sorted(NARROW))
@pytest.mark.parametrize("case", [(2, 14, 13, 64, 128, 4, 2, 1), (1, 23, 21, 128, 72, 3, 2, 1), (3, 9, 30, 192, 136, 2, 2, 0), (2, 11, 10, 64, 40, 5, 3, 2)])
@pytest.mark.parametrize("out_dtype", ["same", "f32"])
def test_conv_transposed(cfg, case, out_dtype):
    n, H, W, Cin, Cout, k, s, p = case
    w = wl.Workload("narrow_convT", "conv", BF16, BF16 if out_dtype == "same" else F32, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout,
                    KH=k, KW=k, stride=(s, s), pad=(p, p), transposed=1, dist_b=("normal", float(np.sqrt(2.0 / (k * k * Cin)))))
    check_full(w, force=f"mfma:{cfg}", expect_kernel=f"{NARROW[cfg]}x128x32")


@pytest.mark.parametrize("M,N,K,trans_b,tile", [
    (3072, 2048, 1024, 0, "128x256x32_w2x4_a64"), (3840, 4096, 648, 0, "256x256x32"), (4097, 4096, 1024, 0, "160x256x32"), (2600, 5120, 1024, 1, "224x256x32"),
    (2600, 4352, 1024, 1, "192x256x32"), (2048, 4096, 1024, 1, "128x256x32_w2x4_a64"),
    (6400, 4096, 2040, 0, "224x256x32"), (6400, 4096, 2048, 0, "256x256x32"), (2600, 5120, 2048, 1, "224x256x32"), (4608, 4864, 2048, 1, "192x256x32"),   # a twelfth less: long, several rounds
])
def test_dispatch(M, N, K, trans_b, tile):
    """One height each of the rule: rounds of 256 tiles times rows + 200."""
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    B = (torch.randn((N, K) if trans_b else (K, N), generator=g, device="cuda") * K ** -0.5).bfloat16()
    out = torch.empty((M, N), device="cuda", dtype=torch.bfloat16)
    st = pbk.pbk_matmul(A, B, out, None, M, N, K, K, K if trans_b else N, N, BF16, BF16, trans_b, 1.0, C.EPI_NONE, torch.cuda.current_stream())
    assert st == 0 and tile in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
    rows = torch.tensor(sorted({0, 127, 128, 159, 160, 191, 192, 223, 224, M // 2, M - 1}), device="cuda")
    ref = A[rows].double() @ (B.double().t().contiguous() if trans_b else B.double())
    assert torch.all((out[rows].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4)


@pytest.mark.parametrize("n,hw,cin,cout,k,transposed,tile", [
    (9, 65, 64, 128, 3, False, "128x128x64"), (22, 56, 64, 128, 3, False, "320x128x32"), (28, 56, 64, 104, 3, False, "384x128x32"), (32, 56, 64, 128, 3, False, "448x128x32"),
    (33, 28, 64, 128, 1, False, "128x128x64"), (24, 28, 128, 128, 4, True, "320x128x32"), (32, 28, 128, 128, 4, True, "448x128x32"), (16, 28, 128, 128, 4, True, "128x128x64"),
])
def test_dispatch_narrow(n, hw, cin, cout, k, transposed, tile):
    """Rows of a tile by the rounds they make; against the kernel without matrix units."""
    import paper_2603_06731_amd as pbk
    w = wl.Workload("narrow_dispatch", "conv", BF16, BF16, C.EPI_BIAS_RELU, n=n, H=hw, W=hw, Cin=cin, Cout=cout, KH=k, KW=k, stride=(2, 2) if transposed or k == 1 else (1, 1),
                    pad=((k - 1) // 2,) * 2, transposed=int(transposed), dist_b=("normal", float(np.sqrt(2.0 / (k * k * cin)))))
    dev = T.upload(wl.make_inputs(w))
    with T.forced_kernel(None):
        st, out = T.run_workload(w, dev)
    assert st == 0 and tile in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
    got = T.to_host_f64(out, w.out_dtype)
    with T.forced_kernel("generic"):
        st, out = T.run_workload(w, dev)
    ref = T.to_host_f64(out, w.out_dtype)
    assert st == 0 and np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-4)


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("out", ["same", "f32"])
@pytest.mark.parametrize("ldr,ldc", [(272, 272), (277, 264)])          # residual in whole 16-byte pieces, one element at a time
def test_residual(cfg, out, ldr, ldc):
    """The shortcut operand through the epilogue's passes, of 7 or 5 blocks of rows."""
    import torch
    import paper_2603_06731_amd as pbk
    M, N, K = 2 * HEIGHT[cfg] - 5, 264, 200
    g = torch.Generator(device="cuda").manual_seed(cfg)
    td, code = (torch.bfloat16, BF16) if out == "same" else (torch.float32, F32)
    A, B = torch.randn(M, K, generator=g, device="cuda").bfloat16(), (torch.randn(K, N, generator=g, device="cuda") * K ** -0.5).bfloat16()
    R, bias = torch.randn(M, ldr, generator=g, device="cuda").to(td), torch.randn(N, generator=g, device="cuda")
    C_ = torch.full((M, ldc), 7.0, device="cuda", dtype=td)
    with T.forced_kernel(f"mfma:{cfg}"):
        st = pbk.pbk_matmul_residual(A, B, C_, bias, R, M, N, K, K, N, ldc, ldr, BF16, code, 0, 0.5, 2.0, C.EPI_BIAS_RELU)
    assert st == 0 and f"{HEIGHT[cfg]}x256x32" in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
    ref = torch.relu(0.5 * (A.double() @ B.double()) + bias.double() + 2.0 * R[:, :N].double())
    # one rounding to the output type (2^-9 of the value in bf16), fp32 sums of 200 terms of order K^-1/2 and three of order one
    assert torch.all((C_[:, :N].double() - ref).abs() <= (2.0 ** -8 if out == "same" else 0.0) * ref.abs() + 1e-5)
    assert torch.all(C_[:, N:] == 7.0)


@pytest.mark.parametrize("cfg", CFGS + sorted(NARROW))
@pytest.mark.parametrize("out", ["same", "f32"])
def test_residual_conv(cfg, out):
    import torch
    import paper_2603_06731_amd as pbk
    n, hw, Cin, Cout = 2, 27, 64, 72
    g = torch.Generator(device="cuda").manual_seed(cfg)
    td, code = (torch.float16, F16) if out == "same" else (torch.float32, F32)
    x, w = torch.randn(n, hw, hw, Cin, generator=g, device="cuda").half(), (torch.randn(3, 3, Cin, Cout, generator=g, device="cuda") * (9 * Cin) ** -0.5).half()
    r, y = torch.randn(n, hw, hw, Cout, generator=g, device="cuda").to(td), torch.empty(n, hw, hw, Cout, device="cuda", dtype=td)
    with T.forced_kernel(f"mfma:{cfg}"):
        st = pbk.pbk_conv2d_nhwc_residual(x, w, y, None, r, n, hw, hw, Cin, Cout, 3, 3, 1, 1, 1, 1, 1, 1, F16, code, 1.0, -0.5, C.EPI_RELU)
    tile = f"{HEIGHT[cfg]}x256x32" if cfg in HEIGHT else f"{NARROW[cfg]}x128x32"
    assert st == 0 and tile in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
    ref = torch.nn.functional.conv2d(x.double().cpu().permute(0, 3, 1, 2), w.double().cpu().permute(3, 2, 0, 1), padding=1).permute(0, 2, 3, 1)
    ref = torch.relu(ref - 0.5 * r.double().cpu())
    # one rounding to the output type (2^-12 of the value in f16), fp32 sums of 576 terms of order one 24th
    assert torch.all((y.double().cpu() - ref).abs() <= (2.0 ** -11 if out == "same" else 0.0) * ref.abs() + 1e-5)
