"""Attention of a few queries with the keys split over workgroups, whose parts meet in a stream's scratch memory: against the
definition in float64, bit-for-bit repetition on one stream and on two at once, and the calls that go without scratch memory."""
import pytest

import workloads as wl
import pbk_testlib as T

pytestmark = pytest.mark.gpu

BF16, F16 = wl.DTYPE_BF16, wl.DTYPE_F16


def operands(b, Nq, Nk, D, dtype, pad=0, seed=0):
    """Rows padded with NaN, one key whose scores move the reference point."""
    import torch
    tdt = torch.bfloat16 if dtype == BF16 else torch.float16
    g = torch.Generator().manual_seed(b * 1000 + Nk + seed)
    q, k, v = (torch.full((b, n, D + pad), float("nan")) for n in (Nq, Nk, Nk))
    for x in (q, k, v):
        x[..., :D] = torch.randn(x[..., :D].shape, generator=g)
    k[:, Nk // 2, :D] *= 6.0
    return [x.to(tdt).cuda() for x in (q, k, v)]


def call(q, k, v, out, D, dtype, causal, stream=None):
    import paper_2603_06731_amd as pbk
    (b, Nq, ld), Nk = q.shape, k.shape[1]
    dims = (b, Nq, Nk, D, ld, ld, ld, ld, Nq * ld, Nk * ld, Nk * ld, Nq * ld)
    if causal:
        return pbk.pbk_attention_causal(q, k, v, out, *dims, dtype, D ** -0.5, stream)
    return pbk.pbk_attention(q, k, v, None, out, *dims, 0, 0, dtype, D ** -0.5, stream)


def close(q, k, v, out, D, dtype, causal):
    import torch
    qd, kd, vd = (x[..., :D].double() for x in (q, k, v))
    Nq, Nk = q.shape[1], k.shape[1]
    s = qd @ kd.transpose(1, 2).contiguous() * D ** -0.5
    if causal:
        s = s.masked_fill(torch.arange(Nk, device=q.device)[None, :] > torch.arange(Nq, device=q.device)[:, None] + Nk - Nq, float("-inf"))
    w = torch.softmax(s, -1)
    ref, got = w @ vd, out[..., :D].double()
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    # weights rounded to 16 bits (u of their value), then the output: u (sum w |v| + |o|), with fp32 sums below that
    u = 2.0 ** -8 if dtype == BF16 else 2.0 ** -11
    return bool(((got - ref).abs() <= u * ((w @ vd.abs()) + ref.abs()) + 1e-5)[~torch.isnan(ref)].all())


CASES = [  # batch, Nq, Nk, row padding
    (3, 16, 33, 8),          # two parts, the second with one key
    (2, 5, 67, 0),           # a last part that no causal query but the last sees
    (96, 1, 64, 0),          # most entries, two parts
    (5, 8, 520, 8),          # parts of one step and of none beyond
    (2, 3, 2050, 0),         # 64 parts, more than are requested together, some with two steps
    (1, 16, 4096, 0),
    (2, 70 - 56, 9, 0),      # more queries than keys: a single step, not split; rows that see none are NaN
]


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_keys_split(D, dtype, causal):
    import torch
    import paper_2603_06731_amd as pbk
    for b, Nq, Nk, pad in CASES:
        q, k, v = operands(b, Nq, Nk, D, dtype, pad)
        out = torch.zeros_like(q)
        with T.forced_kernel("decode:8"):
            assert call(q, k, v, out, D, dtype, causal) == 0
        assert ("split" in pbk.pbk_last_kernel()) == (Nk > 32)
        assert torch.all(out[..., D:] == 0)
        assert close(q, k, v, out, D, dtype, causal), (b, Nq, Nk)


@pytest.mark.parametrize("batch,Nk,D,split", [
    (16, 1535, 128, False), (16, 1536, 128, True), (64, 2559, 64, False), (64, 2560, 64, True), (33, 3583, 32, False), (33, 3584, 32, True),
    (65, 4095, 128, False), (65, 4096, 64, True), (96, 4096, 32, True), (97, 4096, 32, False), (1, 40000, 32, True)])
def test_dispatch(batch, Nk, D, split):
    """Either side of each line of the rule, with the automatic choice."""
    import torch
    import paper_2603_06731_amd as pbk
    q, k, v = operands(batch, 1, Nk, D, BF16)
    out = torch.empty_like(q)
    with T.forced_kernel(None):
        assert call(q, k, v, out, D, BF16, 1) == 0
    assert ("split" in pbk.pbk_last_kernel()) == split, pbk.pbk_last_kernel()
    assert close(q, k, v, out, D, BF16, 1)


def test_repeats_and_streams():
    """The same bits call after call, with the parts arriving in any order, while another stream does the same with other operands."""
    import torch
    a, b = (operands(12, 4, 4096, 128, BF16, seed=s) for s in (1, 2))
    oa, ob = [torch.empty_like(a[0]) for _ in range(24)], [torch.empty_like(b[0]) for _ in range(24)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for x, y in zip(oa, ob):
        assert call(*a, x, 128, BF16, 1, streams[0]) == 0 and call(*b, y, 128, BF16, 1, streams[1]) == 0
    torch.cuda.synchronize()
    assert close(*a, oa[0], 128, BF16, 1) and close(*b, ob[0], 128, BF16, 1)
    assert all(torch.equal(x, oa[0]) for x in oa) and all(torch.equal(y, ob[0]) for y in ob)


def test_without_scratch_memory():
    """A captured call goes without a split and replays next to eager ones; released memory is obtained again."""
    import torch
    import paper_2603_06731_amd as pbk
    q, k, v = operands(8, 2, 4096, 128, BF16)
    out, cap = torch.empty_like(q), torch.empty_like(q)
    assert call(q, k, v, out, 128, BF16, 1, torch.cuda.current_stream()) == 0 and "split" in pbk.pbk_last_kernel()
    eager = out.clone()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        assert call(q, k, v, cap, 128, BF16, 1, torch.cuda.current_stream()) == 0
        assert "split" not in pbk.pbk_last_kernel() and "decode" in pbk.pbk_last_kernel()
    for _ in range(3):
        cap.zero_()
        graph.replay()
        assert call(q, k, v, out, 128, BF16, 1, torch.cuda.current_stream()) == 0
        torch.cuda.synchronize()
        assert torch.equal(out, eager) and close(q, k, v, cap, 128, BF16, 1)
    assert pbk.pbk_release_scratch() == 0
    out.zero_()
    assert call(q, k, v, out, 128, BF16, 1, torch.cuda.current_stream()) == 0 and "split" in pbk.pbk_last_kernel()
    assert torch.equal(out, eager)
