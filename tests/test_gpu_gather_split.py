"""The gathering kernel with eight waves and k-tiles of 64, and with the k-tiles split over workgroups: against the oracle, at the edges of its
rules, bit-for-bit repetition, and captured."""
import numpy as np
import pytest

import workloads as wl
from workloads import configs as C
import pbk_testlib as T
from test_gpu_bstat import run_case
from test_gpu_few_tiles import TOL

pytestmark = pytest.mark.gpu

BF16, F16, F32 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32


@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("dtype,out_dtype,epi", [(BF16, BF16, C.EPI_BIAS_GELU_TANH), (F16, F16, C.EPI_BIAS_RELU), (BF16, F32, C.EPI_NONE)])
@pytest.mark.parametrize("batch,M,N,K,kernel", [
    (1, 64, 129, 704, "64x128x64_w4x2"),        # eleven k-tiles: not split
    (1, 65, 129, 705, "64x128x64_w4x2_split"),  # twelve: two parts; a second row tile with one row
    (2, 5, 131, 1601, "64x128x64_w4x2_split"),  # four parts of six or seven k-tiles, waves without rows, batches
    (1, 33, 77, 5123, "64x128x64_w4x2_split"),  # eight parts
    (1, 4096, 255, 1000, "64x128x64_w4x2_split"),    # 128 tiles
    (1, 4097, 255, 1000, "64x128x64_w4x2"),     # 130
    (1, 8192, 255, 300, "64x128x64_w4x2"),      # 256: one per compute unit
    (1, 8193, 255, 300, "64x128x32_w2x2"),      # more
])
def test_matmul(batch, M, N, K, kernel, dtype, out_dtype, epi, trans_b):
    err, kern = run_case(batch, M, N, K, dtype, out_dtype, trans_b, epi, pad_ld=1, force=None, bias_on=epi != C.EPI_NONE)
    assert kern.endswith(kernel), kern
    assert err <= TOL[out_dtype], err


CONVS = [  # n, H, W, Cin, Cout, KH, KW, stride, pad, dil, split
    (1, 9, 9, 127, 40, 3, 3, (1, 1), (1, 1), (1, 1), True),       # Cin = 127: the last piece of a tap is read early
    (2, 11, 8, 61, 33, 3, 2, (2, 1), (1, 0), (1, 2), False),      # six k-tiles; odd Cout, dilation
    (1, 12, 10, 9, 64, 7, 7, (1, 2), (3, 3), (1, 1), True),       # taps shorter than a k-tile: several begin in each
    (1, 20, 20, 3, 32, 5, 5, (1, 1), (2, 2), (1, 1), False),      # fewer channels than a piece: everything careful
    (3, 7, 7, 100, 130, 5, 5, (1, 1), (2, 2), (1, 1), True),      # images inside a tile, a second column tile
    (1, 18, 18, 61, 32, 7, 7, (2, 2), (0, 0), (1, 1), True),      # a few outputs and a long contraction
]


@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("case", CONVS)
def test_conv(case, dtype):
    import paper_2603_06731_amd as pbk
    n, H, W, Cin, Cout, KH, KW, stride, pad, dil, split = case
    w = wl.Workload("gather_split_conv", "conv", dtype, dtype, C.EPI_BIAS_RELU, n=n, H=H, W=W, Cin=Cin, Cout=Cout, KH=KH, KW=KW,
                    stride=stride, pad=pad, dil=dil, dist_b=("normal", float(np.sqrt(2.0 / (KH * KW * Cin)))))
    host = wl.make_inputs(w)
    st, out = T.run_workload(w, T.upload(host))
    name = pbk.pbk_last_kernel()
    assert st == 0 and "gather_64x128x64" in name and ("split" in name) == split, name
    ref, pre = T.oracle_full(w, host)
    err = T.rel_err(T.to_host_f64(out, w.out_dtype).reshape(ref.shape), ref, pre)
    assert err <= TOL[dtype], err


def test_repeats_residual_and_capture():
    """The same bits call after call, with the parts arriving in any order; a captured call goes without a split."""
    import torch
    import paper_2603_06731_amd as pbk
    M, N, K = 70, 259, 4099
    g = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    b = (torch.randn(K, N, generator=g, device="cuda") * K ** -0.5).bfloat16()
    r = torch.randn(M, N, generator=g, device="cuda").bfloat16()
    outs = [torch.empty(M, N, dtype=torch.bfloat16, device="cuda") for _ in range(16)]

    def call(out):
        return pbk.pbk_matmul_residual(a, b, out, None, r, M, N, K, K, N, N, N, BF16, BF16, 0, 1.0, 2.0, 0, torch.cuda.current_stream())
    ref = a.double() @ b.double() + 2.0 * r.double()
    for x in outs:
        assert call(x) == 0 and "split" in pbk.pbk_last_kernel()
    assert all(torch.equal(x, outs[0]) for x in outs)
    # one rounding to bf16 (2^-9 of the value), fp32 sums of K terms of order K^-1/2
    assert torch.all((outs[0].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4)
    cap, graph = torch.empty_like(outs[0]), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        assert call(cap) == 0 and "split" not in pbk.pbk_last_kernel()
    for _ in range(3):
        cap.zero_()
        graph.replay()
        assert call(outs[1]) == 0
        torch.cuda.synchronize()
        assert torch.equal(outs[1], outs[0])
        assert torch.all((cap.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4)
