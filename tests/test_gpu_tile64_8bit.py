"""64-wide tiles with 8-bit operands: int8 codes bit-exact and FP8 inside the arithmetic bars, both layouts of B, convolutions, every form of the
quantised epilogue, the contraction split over workgroups; and which problems take them."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
from test_gpu_int8 import params, run_matmul, dev_or_none, INT8, F32
from test_gpu_parity import check_full

pytestmark = pytest.mark.gpu

BF16, F16, E4M3, E5M2 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_FP8_E4M3, wl.DTYPE_FP8_E5M2
FORMS = ["tile64:1", "tile64:8"]
SHAPES = [(1, 16, 16), (33, 48, 80), (64, 64, 256), (65, 144, 272), (130, 80, 1040), (31, 32, 2320)]      # pieces, ragged rounds, more rounds than stages


@pytest.mark.parametrize("force", FORMS)
@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("mnk", SHAPES)
def test_int8_matmul(mnk, trans_b, force):
    import oracle
    m, n, k = mnk
    n += trans_b * 5                                    # k-major B: any N
    A, B, q = wl.int8_tensor((m, k), 1), wl.int8_tensor((n, k) if trans_b else (k, n), 2), params(n, 3)
    got, kernel = run_matmul(A, B, q, trans_b, True, force)
    assert "mfma8_tile64" in kernel, kernel
    assert np.array_equal(got, oracle.matmul_int8(A, B, trans_b=trans_b, **q))


@pytest.mark.parametrize("variant", range(6))
@pytest.mark.parametrize("out_int8", [True, False])
@pytest.mark.parametrize("step", [0.043, 2.0 ** -70])   # the second: steps that need the real division
def test_int8_epilogue(variant, out_int8, step):
    import oracle
    m, n, k = 70, 80, 304
    A, B, q = wl.int8_tensor((m, k), 1, "normal", 40.0), wl.int8_tensor((n, k), 2, "normal", 30.0), params(n, variant)
    q["out_scale"] = step
    got, kernel = run_matmul(A, B, q, 1, out_int8, "tile64")
    want = oracle.matmul_int8(A, B, trans_b=1, out_int8=out_int8, **q)
    view = np.uint8 if out_int8 else np.uint32
    assert "tile64" in kernel and np.array_equal(got.view(view), want.view(view)), kernel


@pytest.mark.parametrize("force", FORMS)
@pytest.mark.parametrize("geom", [(2, 15, 14, 32, 48, 3, 1, 1), (1, 9, 11, 16, 16, 3, 2, 1), (3, 7, 7, 256, 80, 1, 2, 0), (1, 8, 8, 80, 144, 5, 1, 2)])
@pytest.mark.parametrize("bn", [False, True])
def test_int8_conv(geom, force, bn):
    import torch
    import oracle
    import paper_2603_06731_amd as pbk
    n, H, W, Cin, Cout, k, s, p = geom
    x, w = wl.int8_tensor((n, H, W, Cin), 1, "normal", 40.0), wl.int8_tensor((k, k, Cin, Cout), 2, "normal", 30.0)
    q = params(Cout, 3)
    r = np.random.default_rng(5)
    mean, var = r.normal(0, 0.3, Cout).astype(np.float32), r.uniform(0.5, 2.0, Cout).astype(np.float32)
    extra = dict(mean=mean, var=var, eps=1e-5) if bn else {}
    if bn:
        q = dict(scale=q["scale"], bias=q["bias"], mid_scale=q["mid_scale"], relu=q["relu"], out_scale=q["out_scale"], gamma=q["mul"], beta=q["add"])
        want = oracle.conv2d_nhwc_int8_bn(x, w, stride=(s, s), pad=(p, p), dil=(1, 1), **extra, **q)
    else:
        want = oracle.conv2d_nhwc_int8(x, w, stride=(s, s), pad=(p, p), dil=(1, 1), **q)
    out = torch.empty(want.size, dtype=torch.int8, device="cuda")
    d = {k2: dev_or_none(v) if isinstance(v, np.ndarray) else v for k2, v in {**q, **extra}.items()}
    args = (torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), out, n, H, W, Cin, Cout, k, k, s, s, p, p, 1, 1, d["scale"], d["bias"], q["mid_scale"])
    with T.forced_kernel(force):
        if bn:
            st = pbk.pbk_conv2d_nhwc_int8_bn(*args, d["mean"], d["var"], 1e-5, d["gamma"], d["beta"], q["relu"], q["out_scale"], INT8, None)
        else:
            st = pbk.pbk_conv2d_nhwc_int8(*args, d["mul"], d["add"], q["relu"], q["out_scale"], INT8, None)
    assert st == 0 and "mfma8_tile64" in pbk.pbk_last_kernel(), (st, pbk.pbk_last_kernel())
    assert np.array_equal(out.cpu().numpy().reshape(want.shape), want)


@pytest.mark.parametrize("force", FORMS)
@pytest.mark.parametrize("dtype,out_dtype,trans_b", [(E4M3, BF16, 1), (E4M3, F16, 0), (E5M2, BF16, 0), (E5M2, F32, 1), (E4M3, F32, 0)])
def test_fp8_matmul(dtype, out_dtype, trans_b, force):
    for m, n, k in SHAPES:
        w = wl.Workload(f"t64_fp8_{m}x{n}x{k}", "matmul", dtype, out_dtype, C.EPI_BIAS_GELU_TANH, alpha=0.5, M=m, N=n + trans_b * 5, K=k, trans_b=trans_b,
                        dist_b=("normal", 1.0 / np.sqrt(k)), dist_bias=("normal", 0.5))
        check_full(w, force=force, expect_kernel="mfma8_tile64")


@pytest.mark.parametrize("force", FORMS)
def test_fp8_conv(force):
    w = wl.Workload("t64_fp8_conv", "conv", E4M3, BF16, C.EPI_BIAS_RELU, n=2, H=13, W=11, Cin=48, Cout=80, KH=3, KW=3, pad=(1, 1), dist_b=("normal", 0.07))
    check_full(w, force=force, expect_kernel="mfma8_tile64")


@pytest.mark.parametrize("dtype,M,N,K,trans_b,tile64", [
    (E4M3, 128, 4096, 3200, 0, True), (E4M3, 128, 4112, 3200, 0, False), (E4M3, 128, 4096, 240, 0, False), (E4M3, 128, 4352, 1024, 1, True),
    (E4M3, 128, 4353, 1024, 1, False), (E4M3, 128, 4353, 2048, 1, True), (E4M3, 128, 6145, 2048, 1, False),
])
def test_dispatch_fp8(dtype, M, N, K, trans_b, tile64):
    """Either side of one tile per compute unit (256 tiles of 32 x 64), of 272 and of 384."""
    w = wl.Workload("t64_dispatch", "matmul", dtype, BF16, C.EPI_BIAS, M=M, N=N, K=K, trans_b=trans_b, dist_b=("normal", 1.0 / np.sqrt(K)))
    check_full(w, expect_kernel="mfma8_tile64" if tile64 else "mfma_128x128")


@pytest.mark.parametrize("m,n,k,tile64", [(256, 4096, 64, True), (256, 4097, 64, False), (128, 4352, 3088, True), (128, 4353, 3088, False)])
def test_dispatch_int8(m, n, k, tile64):
    import oracle
    A, B, q = wl.int8_tensor((m, k), 1), wl.int8_tensor((n, k), 2), params(n, 3)
    got, kernel = run_matmul(A, B, q, 1, True, None)
    assert ("tile64" in kernel) == tile64, kernel
    assert np.array_equal(got, oracle.matmul_int8(A, B, trans_b=1, **q))


@pytest.mark.parametrize("force", ["tile64:0", "tile64:2"])
def test_forms_that_are_not_built(force):
    """64 x 64 tiles are built for the 16-bit types: refused, and nothing is launched."""
    import torch
    import paper_2603_06731_amd as pbk
    m, n, k = 64, 64, 256
    a, b = (torch.ones(r, k, dtype=torch.int8, device="cuda") for r in (m, n))
    out, scale = torch.full((m, n), 7, dtype=torch.int8, device="cuda"), torch.ones(n, device="cuda")
    with T.forced_kernel(force):
        st = pbk.pbk_matmul_int8(a, b, out, m, n, k, k, k, n, 1, scale, None, 0.0, None, None, 0, 1.0, INT8)
        assert "not supported" in pbk.pbk_status_string(st), st
        o = torch.full((m, n), 7.0, device="cuda")
        st = pbk.pbk_matmul(a.view(torch.uint8), b.view(torch.uint8), o, None, m, n, k, k, k, n, E4M3, F32, 1, 1.0, C.EPI_NONE)
        assert "not supported" in pbk.pbk_status_string(st), st
    assert bool((out == 7).all()) and bool((o == 7).all())


@pytest.mark.parametrize("M,N,K,split", [(64, 512, 3056, True), (64, 512, 2816, False), (128, 2304, 8192, True), (128, 2304, 5888, False), (128, 2816, 8192, False)])
def test_dispatch_split_fp8(M, N, K, split):
    """16 tiles, 12 rounds of 256 and 11; 144 tiles, 32 and 23 (24); 176."""
    import paper_2603_06731_amd as pbk
    w = wl.Workload("t64_split_dispatch", "matmul", E4M3, BF16, C.EPI_BIAS, M=M, N=N, K=K, trans_b=1, dist_b=("normal", 1.0 / np.sqrt(K)))
    check_full(w, expect_kernel="mfma8_tile64")
    assert pbk.pbk_last_kernel().endswith("_split") == split, pbk.pbk_last_kernel()


@pytest.mark.parametrize("M,N,K,split", [(1, 1408, 4096, True), (8, 1408, 3536, False), (8, 1408, 3568, True), (2, 2000, 3056, False), (2, 2000, 3072, True)])
def test_dispatch_split_few_rows_fp8(M, N, K, split):
    """Up to 16 rows over a row-major B: five million values of B, and K = 3072."""
    import paper_2603_06731_amd as pbk
    w = wl.Workload("t64_split_few_rows", "matmul", E4M3, BF16, C.EPI_BIAS, M=M, N=N, K=K, dist_b=("normal", 1.0 / np.sqrt(K)))
    check_full(w, expect_kernel="mfma8_tile64")
    assert pbk.pbk_last_kernel().endswith("_split") == split, pbk.pbk_last_kernel()


@pytest.mark.parametrize("m,n,k,split", [(64, 512, 3056, True), (64, 512, 2816, False), (128, 2304, 8192, True), (128, 2304, 5888, False)])
def test_dispatch_split_int8(m, n, k, split):
    import oracle
    A, B, q = wl.int8_tensor((m, k), 1), wl.int8_tensor((n, k), 2), params(n, 3)
    got, kernel = run_matmul(A, B, q, 1, True, None)
    assert "mfma8_tile64" in kernel and kernel.endswith("_split") == split, kernel
    assert np.array_equal(got, oracle.matmul_int8(A, B, trans_b=1, **q))


@pytest.mark.parametrize("trans_b", [0, 1])
def test_forced_split_is_one(trans_b):
    """"tile64:8" splits whatever has two rounds of 256 values of k, and the other form never does."""
    import oracle
    for m, n, k in SHAPES:
        n += trans_b * 5
        A, B, q = wl.int8_tensor((m, k), 1), wl.int8_tensor((n, k) if trans_b else (k, n), 2), params(n, 3)
        for force in FORMS:
            got, kernel = run_matmul(A, B, q, trans_b, True, force)
            assert kernel.endswith("_split") == (force == "tile64:8" and k > 256), (kernel, k)
            assert np.array_equal(got, oracle.matmul_int8(A, B, trans_b=trans_b, **q))
