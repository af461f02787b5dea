"""Run-to-run equality, bit by bit, of the kernels that split a contraction or the keys over waves (their partial results are added in
a fixed order) and of the kernels beside them: the same call sixteen times over, with the output poisoned in between."""
import pytest

import workloads as wl
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16 = wl.DTYPE_BF16


def repeats(call, out, force, name):
    import torch
    import paper_2603_06731_amd as pbk
    first = None
    with T.forced_kernel(force):
        for _ in range(16):
            out.fill_(float("nan"))
            assert call() == 0 and name in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
            bits = out.view(torch.int16).clone()
            first = bits if first is None else first
            assert torch.equal(bits, first)
    assert not bool(torch.isnan(out).any())


@pytest.mark.parametrize("force,name", [("ksplit:0", "16x64"), ("ksplit:1", "16x32"), ("tile64:0", "64x64_s4"), ("tile64:1", "32x64_s3"), ("tile64:2", "64x64_s2"),
                                        ("mfma:2", "w2x4_s4"), ("gather:0", "gather_128"), ("gather:1", "gather_64")])
def test_matmul(force, name):
    import torch
    import paper_2603_06731_amd as pbk
    M, N, K = (16, 4096, 4104) if "ksplit" in force else (577, 1032, 2056)
    g = torch.Generator(device="cuda").manual_seed(7)
    a, b = (torch.randn(*s, generator=g, device="cuda").bfloat16() for s in ((M, K), (K, N)))
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    repeats(lambda: pbk.pbk_matmul(a, b, out, None, M, N, K, K, N, N, BF16, BF16, 0, 1.0, 0), out, force, name)


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("force,name,batch,Nq,Nk,D", [
    ("decode:1", "decode", 64, 7, 1111, 64), ("decode:2", "decode", 64, 16, 1111, 128), ("decode:4", "decode", 16, 1, 8192, 128),
    ("mfma:2", "kv64x2", 16, 1025, 1111, 64), ("mfma:2", "kv64x2", 4, 1025, 2048, 128), ("mfma:2", "kv64x2", 16, 500, 1111, 32)])
def test_attention(force, name, batch, Nq, Nk, D, causal):
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(8)
    q, k, v = (torch.randn(batch, n, D, generator=g, device="cuda").bfloat16() for n in (Nq, Nk, Nk))
    out = torch.empty_like(q)
    dims = (batch, Nq, Nk, D, D, D, D, D, Nq * D, Nk * D, Nk * D, Nq * D)

    def call():
        if causal:
            return pbk.pbk_attention_causal(q, k, v, out, *dims, BF16, D ** -0.5)
        return pbk.pbk_attention(q, k, v, None, out, *dims, 0, 0, BF16, D ** -0.5)
    repeats(call, out, force, name)


@pytest.mark.parametrize("force,name", [("mfma:1", "w2x4_s2"), ("mfma:2", "w2x4_s4"), ("mfma:6", "128x256")])
def test_transposed_convolution(force, name):
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn(8, 28, 28, 264, generator=g, device="cuda").bfloat16()
    w = torch.randn(4, 4, 264, 136, generator=g, device="cuda").bfloat16()
    out = torch.empty(8, 56, 56, 136, dtype=torch.bfloat16, device="cuda")
    repeats(lambda: pbk.pbk_conv2d_transpose_nhwc(x, w, out, None, 8, 28, 28, 264, 136, 4, 4, 2, 2, 1, 1, 0, 0, 1, 1, BF16, BF16, 1.0, 0), out, force, name)


@pytest.mark.parametrize("M,N,K,trans_b,name", [
    (577, 1024, 4096, 0, "tile64_64x64_s2_split"), (513, 1080, 3336, 1, "tile64_64x64_s2_split"), (128, 2304, 6144, 0, "tile64_32x64_s3_split"),
    (2600, 5120, 1024, 1, "224x256x32"), (4097, 4096, 1024, 0, "160x256x32"),
])
def test_matmul_automatic(M, N, K, trans_b, name):
    import torch
    import paper_2603_06731_amd as pbk
    g = torch.Generator(device="cuda").manual_seed(7)
    a, b = (torch.randn(*s, generator=g, device="cuda").bfloat16() for s in ((M, K), (N, K) if trans_b else (K, N)))
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    repeats(lambda: pbk.pbk_matmul(a, b, out, None, M, N, K, K, K if trans_b else N, N, BF16, BF16, trans_b, 1.0, 0), out, None, name)


@pytest.mark.parametrize("name", ["tile64_32x64_s3_split"])
def test_fp8_split(name):
    import torch
    import paper_2603_06731_amd as pbk
    M, N, K = 128, 2304, 8192
    g = torch.Generator(device="cuda").manual_seed(7)
    a, b = (torch.randn(r, K, generator=g, device="cuda").to(torch.float8_e4m3fn).view(torch.uint8) for r in (M, N))
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    repeats(lambda: pbk.pbk_matmul(a, b, out, None, M, N, K, K, K, N, wl.DTYPE_FP8_E4M3, BF16, 1, 1.0, 0), out, None, name)


@pytest.mark.parametrize("force,name", [("mfma:14", "256x128x32"), ("mfma:15", "320x128x32"), ("mfma:16", "384x128x32"), ("mfma:17", "448x128x32"), (None, "tile64_32x64_s3_classes")])
def test_transposed_convolution_tall(force, name):
    import torch
    import paper_2603_06731_amd as pbk
    n, hw = (8, 28) if force else (2, 14)
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn(n, hw, hw, 256, generator=g, device="cuda").bfloat16()
    w = torch.randn(4, 4, 256, 136, generator=g, device="cuda").bfloat16()
    out = torch.empty(n, 2 * hw, 2 * hw, 136, dtype=torch.bfloat16, device="cuda")
    repeats(lambda: pbk.pbk_conv2d_transpose_nhwc(x, w, out, None, n, hw, hw, 256, 136, 4, 4, 2, 2, 1, 1, 0, 0, 1, 1, BF16, BF16, 1.0, 0), out, force, name)


@pytest.mark.parametrize("force", ["gather:0", "gather:1", "gather:4", None])
def test_rows_of_taps(force):
    """... and, by the automatic choice, in three parts."""
    import torch
    import paper_2603_06731_amd as pbk
    n, hw, Cin, Cout, k = (4, 40, 11, 72, 7) if force else (1, 20, 11, 72, 7)
    g = torch.Generator(device="cuda").manual_seed(11)
    x, w = torch.randn(n, hw, hw, Cin, generator=g, device="cuda").bfloat16(), torch.randn(k, k, Cin, Cout, generator=g, device="cuda").bfloat16()
    out = torch.empty(n, hw, hw, Cout, dtype=torch.bfloat16, device="cuda")
    repeats(lambda: pbk.pbk_conv2d_nhwc(x, w, out, None, n, hw, hw, Cin, Cout, k, k, 1, 1, 3, 3, 1, 1, BF16, BF16, 1.0, 0), out, force, "rows_gather" if force else "_split")
