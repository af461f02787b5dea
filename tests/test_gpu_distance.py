"""Distance from 64 bits of the kernels that split a contraction or the keys of an attention over waves or workgroups, beside that of the
kernel that walks it in one piece: relative 2-norm over some problems of the sizes that the automatic choice gives them.

A split changes the order of fp32 sums and, for attention, which power of two the 16-bit weights are scaled by.  Neither may cost
precision.  The bound: the ratio of the two distances is a ratio of two sample deviations over n >= 2e5 rounding errors,
whose standard deviation is below 1 / sqrt(n) = 0.0023; 1.01 is more than four of them.  For the products both distances are
those of one and the same rounding of the output."""
import pytest

import workloads as wl
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16, F16, F32 = wl.DTYPE_BF16, wl.DTYPE_F16, wl.DTYPE_F32


class Distance:
    def __init__(self):
        self.d2, self.r2, self.n = 0.0, 0.0, 0

    def add(self, got, ref):
        self.d2 += float((got.double() - ref).pow(2).sum())
        self.r2 += float(ref.pow(2).sum())
        self.n += ref.numel()

    def rel(self):
        return (self.d2 / self.r2) ** 0.5


def compare(problems, before, now, name):
    """problems: generator of (call(out_forced_choice) -> output tensor, float64 reference)."""
    import paper_2603_06731_amd as pbk
    dist = {before: Distance(), now: Distance()}
    for call, ref in problems:
        for force in (before, now):
            with T.forced_kernel(force):
                out = call()
            if force == now:
                assert name in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
            else:
                assert name not in pbk.pbk_last_kernel(), pbk.pbk_last_kernel()
            dist[force].add(out, ref)
    assert dist[now].n >= 2e5
    ratio = dist[now].rel() / dist[before].rel()
    print(f"{name}: {dist[before].rel():.4e} -> {dist[now].rel():.4e} ratio {ratio:.4f} over {dist[now].n} values", flush=True)
    assert ratio <= 1.01, ratio


def gen(seed):
    import torch
    return torch.Generator(device="cuda").manual_seed(seed)


def types(dtype):
    import torch
    return {BF16: torch.bfloat16, F16: torch.float16, F32: torch.float32}[dtype]


def attention_problems(sizes, dtype, causal):
    import torch
    import paper_2603_06731_amd as pbk
    for seed, (b, Nq, Nk, D) in enumerate(sizes):
        g = gen(seed)
        q, k, v = (torch.randn(b, n, D, generator=g, device="cuda").to(types(dtype)) for n in (Nq, Nk, Nk))
        dims = (b, Nq, Nk, D, D, D, D, D, Nq * D, Nk * D, Nk * D, Nq * D)

        def call():
            out = torch.empty_like(q)
            if causal:
                st = pbk.pbk_attention_causal(q, k, v, out, *dims, dtype, D ** -0.5)
            else:
                st = pbk.pbk_attention(q, k, v, None, out, *dims, 0, 0, dtype, D ** -0.5)
            assert st == 0
            return out
        ref = torch.empty(b, Nq, D, dtype=torch.float64, device="cuda")
        hidden = torch.arange(Nk, device="cuda")[None, :] > torch.arange(Nq, device="cuda")[:, None] + Nk - Nq
        for i in range(b):
            s = q[i].double() @ k[i].double().T * D ** -0.5
            ref[i] = torch.softmax(s.masked_fill(hidden, float("-inf")) if causal else s, -1) @ v[i].double()
        yield call, ref


@pytest.mark.parametrize("dtype", [BF16, F16])
def test_attention_few_queries(dtype):
    sizes = [(128, 8, 128, 64), (128, 8, 1000, 64), (200, 4, 512, 64), (128, 8, 300, 128), (200, 8, 2048, 128), (64, 1, 8192, 128),
             (256, 1, 1024, 128), (256, 16, 500, 32)]
    compare(attention_problems(sizes, dtype, 1), "mfma:1", "decode", "decode")


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("dtype", [BF16, F16])
def test_attention_two_groups(dtype, causal):
    sizes = [(8, 1024, 1024, 64), (6, 2048, 2048, 64), (4, 2000, 2000, 128), (16, 1024, 1024, 32)]
    compare(attention_problems(sizes, dtype, causal), "mfma:1", "mfma:2", "kv64x2")


@pytest.mark.parametrize("dtype", [BF16, F16])
def test_attention_keys_over_workgroups(dtype):
    sizes = [(96, 16, 4096, 128), (64, 8, 2560, 64), (16, 16, 8192, 128), (33, 8, 3584, 32), (24, 4, 5000, 64)]
    compare(attention_problems(sizes, dtype, 1), "decode:4", "decode:8", "split")


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("now,name", [("mfma:3", "q64_kv64x2"), ("mfma:4", "q64_kv64x4")])
def test_attention_64_queries(now, name, dtype, causal):
    sizes = [(16, 577, 577, 64), (8, 2048, 2048, 64), (12, 1024, 1024, 32)] + ([(16, 300, 1024, 128)] if now == "mfma:3" else [])
    compare(attention_problems(sizes, dtype, causal), "mfma:1", now, name)


def matmul_problems(sizes, dtype):
    import torch
    import paper_2603_06731_amd as pbk
    for seed, (M, N, K, t) in enumerate(sizes):
        g = gen(seed)
        A = torch.randn(M, K, generator=g, device="cuda").to(types(dtype))
        W = (torch.randn(*((N, K) if t else (K, N)), generator=g, device="cuda") * K ** -0.5).to(types(dtype))

        def call():
            out = torch.empty(M, N, dtype=types(dtype), device="cuda")
            assert pbk.pbk_matmul(A, W, out, None, M, N, K, K, K if t else N, N, dtype, dtype, t, 1.0, 0) == 0
            return out
        Wd = W.double()
        yield call, A.double() @ (Wd.T.contiguous() if t else Wd)


@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("now,name", [("ksplit", "ksplit"), ("tile64:0", "tile64_64x64_s4"), ("tile64:1", "tile64_32x64"), ("tile64:2", "tile64_64x64_s2")])
def test_matmul(dtype, now, name):
    sizes = [(16, 4096, 4096, 0), (8, 14336, 1024, 0), (16, 2048, 512, 1), (9, 4096, 8192, 1)] if now == "ksplit" else [
        (577, 1024, 1024, 0), (300, 512, 4096, 1), (256, 512, 512, 0)]
    compare(matmul_problems(sizes, dtype), "mfma:1", now, name)


@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("before,now,name", [("tile64:1", "tile64:8", "split"), ("gather:0", "gather:1", "split")])
def test_matmul_over_workgroups(dtype, before, now, name):
    odd = 3 if now == "gather:1" else 0
    compare(matmul_problems([(256, 1024, 4096 + odd, 0), (48, 1024, 16384 + odd, 1), (130, 1000, 1536 + odd, 1)], dtype), before, now, name)


@pytest.mark.parametrize("before", ["mfma:1", "generic"])
def test_f32(before):
    """k over the waves of a tile: partial sums of K / waves terms, no further from 64 bits than one sum of K."""
    compare(matmul_problems([(256, 256, 256, 0), (128, 160, 1024, 1), (512, 512, 512, 0), (800, 800, 320, 1)], F32), before, "small", "small_f32")


@pytest.mark.parametrize("now", ["tile64:0", "tile64:1"])
def test_convolution(now):
    import torch
    import paper_2603_06731_amd as pbk

    def problems():
        for seed, (n, hw, ci, co, k, s) in enumerate([(8, 14, 256, 128, 3, 1), (2, 28, 64, 96, 3, 2), (4, 14, 512, 64, 1, 2)]):
            g = gen(seed)
            x = torch.randn(n, hw, hw, ci, generator=g, device="cuda").bfloat16()
            w = (torch.randn(k, k, ci, co, generator=g, device="cuda") * (k * k * ci) ** -0.5).bfloat16()
            p = k // 2
            oh = (hw + 2 * p - k) // s + 1

            def call():
                y = torch.empty(n, oh, oh, co, dtype=torch.bfloat16, device="cuda")
                assert pbk.pbk_conv2d_nhwc(x, w, y, None, n, hw, hw, ci, co, k, k, s, s, p, p, 1, 1, BF16, BF16, 1.0, 0) == 0
                return y
            cols = torch.nn.functional.unfold(x.double().permute(0, 3, 1, 2).contiguous().cpu(), k, padding=p, stride=s)
            ref = w.double().permute(3, 2, 0, 1).reshape(co, -1).cpu() @ cols
            yield call, ref.reshape(n, co, oh, oh).permute(0, 2, 3, 1).cuda()
    compare(problems(), "mfma:1", now, "tile64")


@pytest.mark.parametrize("dtype", [BF16, F16])
def test_few_rows_f32_results(dtype):
    """Up to 16 rows over a row-major B with fp32 results: the automatic choice is no further from 64 bits than sixteen sums of k / 16 values."""
    import torch
    import paper_2603_06731_amd as pbk
    for M, N, K in [(8, 14336, 4096), (16, 13184, 4992), (5, 8256, 2048), (16, 8192, 4096), (8, 5504, 6144), (3, 8200, 5640), (8, 4096, 14336), (16, 1024, 4888)]:
        dist = {f: Distance() for f in ("ksplit", None)}
        for seed in range(-(-200000 // (M * N))):
            g = gen(seed)
            A = torch.randn(M, K, generator=g, device="cuda").to(types(dtype))
            B = (torch.randn(K, N, generator=g, device="cuda") * K ** -0.5).to(types(dtype))
            ref = A.double() @ B.double()
            for force in dist:
                out = torch.empty(M, N, device="cuda")
                with T.forced_kernel(force):
                    assert pbk.pbk_matmul(A, B, out, None, M, N, K, K, N, N, dtype, F32, 0, 1.0, 0) == 0
                dist[force].add(out, ref)
        ratio = dist[None].rel() / dist["ksplit"].rel()
        print(M, N, K, pbk.pbk_last_kernel(), f"{dist['ksplit'].rel():.3e} {ratio:.4f}", flush=True)
        assert dist[None].n >= 2e5 and ratio <= 1.01, (M, N, K, ratio)
