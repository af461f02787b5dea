"""Sizes at which the choice between kernels has changed sides: what the call gives there, with the automatic choice and whichever kernel that takes.  (Which
one it is stands in the dispatch tests of the kernels.)"""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
from test_gpu_few_tiles import TOL
from test_gpu_tile64_split import call, product, reference

pytestmark = pytest.mark.gpu

BF16, E4M3 = wl.DTYPE_BF16, wl.DTYPE_FP8_E4M3


@pytest.mark.parametrize("dtype,M,N,K,trans_b", [
    (BF16, 2049, 4096, 512, 0), (BF16, 2048, 4096, 4096, 0), (BF16, 4097, 4096, 768, 0),
    (BF16, 2049, 4096, 504, 1), (BF16, 2048, 4096, 1024, 1), (E4M3, 2048, 4096, 512, 1),
])
def test_two_tiles_per_unit(dtype, M, N, K, trans_b):
    import torch
    import paper_2603_06731_amd as pbk
    tdt = torch.bfloat16 if dtype == BF16 else torch.float8_e4m3fn
    g = torch.Generator(device="cuda").manual_seed(7)
    A = torch.randn(M, K, generator=g, device="cuda").to(tdt)
    B = torch.randn(*((N, K) if trans_b else (K, N)), generator=g, device="cuda").to(tdt)
    out = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
    raw = (lambda x: x) if dtype == BF16 else (lambda x: x.view(torch.uint8))
    with T.forced_kernel(None):
        assert pbk.pbk_matmul(raw(A), raw(B), out, None, M, N, K, K, K if trans_b else N, N, dtype, BF16, trans_b, 1.0, C.EPI_NONE) == 0
    a, b = A.double(), B.double().t().contiguous() if trans_b else B.double()
    ref = a @ b
    # rounded once to bf16; the sums in fp32 (FP8: the instruction's own, 1e-4 to 2e-4 of the output's scale)
    bound = 2.0 ** -8 * ref.abs() + (4e-4 if dtype == E4M3 else 1e-5) * K ** 0.5 + 1e-5 * (a.abs() @ b.abs())
    assert torch.all((out.double() - ref).abs() <= bound)


@pytest.mark.parametrize("M,N,K,trans_b", [(257, 1024, 4096, 1), (16, 1024, 5856, 0), (16, 8256, 4096, 0), (513, 1024, 3072, 0)])
def test_few_tiles(M, N, K, trans_b):
    import torch
    a, b = product(M, N, K, trans_b)
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    with T.forced_kernel(None):
        assert call(a, b, out, trans_b) == 0
    ref = reference(a, b, trans_b)
    # one rounding to bf16 (2^-9 of the value), fp32 sums of K terms of order K^-1/2
    assert torch.all((out.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4)


@pytest.mark.parametrize("n,Cin", [(4, 128), (8, 128), (8, 144), (8, 152)])
def test_few_tiles_conv(n, Cin):
    w = wl.Workload("former_line_conv", "conv", BF16, BF16, C.EPI_BIAS_RELU, n=n, H=14, W=14, Cin=Cin, Cout=128, KH=3, KW=3, pad=(1, 1),
                    dist_b=("normal", float(np.sqrt(2.0 / (9 * Cin)))))
    host = wl.make_inputs(w)
    with T.forced_kernel(None):
        st, out = T.run_workload(w, T.upload(host))
    assert st == 0
    ref, pre = T.oracle_full(w, host)
    err = T.rel_err(T.to_host_f64(out, w.out_dtype).reshape(ref.shape), ref, pre)
    assert err <= TOL[BF16], err
