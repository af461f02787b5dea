"""Scratch memory and many streams: more of them than there is memory for, busy and idle, streams that come and go with work under way, and
calls next to a capture."""
import ctypes

import pytest

import test_gpu_tile64_split as S
import workloads as wl

pytestmark = pytest.mark.gpu

BF16 = wl.DTYPE_BF16
M, N, K = 48, 1024, 4096


class Streams:
    """Streams straight from the runtime (torch's pool holds 32 and destroys none)."""

    def __init__(self):
        with open("/proc/self/maps") as f:
            path = next(line.split()[-1] for line in f if "libamdhip64" in line)
        self.hip = ctypes.CDLL(path)

    def create(self):
        s = ctypes.c_void_p()
        assert self.hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
        return s.value

    def destroy(self, s):
        assert self.hip.hipStreamDestroy(ctypes.c_void_p(s)) == 0


@pytest.fixture
def problem():
    import torch
    import paper_2603_06731_amd as pbk
    a, b = S.product(M, N, K)
    ref = S.reference(a, b)

    def good(out):
        return bool(torch.all((out.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4))
    x = torch.randn(4096, 4096, device="cuda").bfloat16()

    def occupy(stream, y, n):                       # some 0.1 ms each
        for _ in range(n):
            pbk.check(pbk.pbk_matmul(x, x, y, None, 4096, 4096, 4096, 4096, 4096, 4096, BF16, BF16, 0, 1.0, 0, stream))
    torch.cuda.synchronize()
    assert pbk.pbk_release_scratch() == 0
    yield a, b, good, occupy
    torch.cuda.synchronize()
    assert pbk.pbk_release_scratch() == 0


def split():
    import paper_2603_06731_amd as pbk
    return pbk.pbk_last_kernel().endswith("_split")


def test_more_streams_than_memory(problem):
    import torch
    a, b, good, occupy = problem
    st = Streams()
    streams = [st.create() for _ in range(40)]
    outs = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in streams]
    ys = [torch.empty(4096, 4096, dtype=torch.bfloat16, device="cuda") for _ in range(32)]
    torch.cuda.synchronize()
    for s, o in zip(streams, outs):                 # one after the other: every stream gets memory
        assert S.call(a, b, o, stream=s) == 0 and split()
        torch.cuda.synchronize()
    assert all(good(o) for o in outs)
    for i in range(32):                             # all of it at work: the next stream goes without
        outs[i].fill_(float("nan"))
    outs[32].fill_(float("nan"))
    torch.cuda.synchronize()
    for i in range(32):
        occupy(streams[i], ys[i], 50)
        assert S.call(a, b, outs[i], stream=streams[i]) == 0
    assert S.call(a, b, outs[32], stream=streams[32]) == 0
    unsplit = not split()
    torch.cuda.synchronize()
    assert unsplit and all(good(o) for o in outs)
    for s in streams:
        st.destroy(s)


def test_streams_that_come_and_go(problem):
    """A stream is destroyed with its work under way and another one is made, often with the same handle."""
    import torch
    a, b, good, occupy = problem
    st = Streams()
    outs = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(60)]
    y = torch.empty(4096, 4096, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    handles = set()
    for i, o in enumerate(outs):
        s = st.create()
        handles.add(s)
        if i % 4 == 0:
            occupy(s, y, 2)
        assert S.call(a, b, o, stream=s) == 0
        st.destroy(s)
    torch.cuda.synchronize()
    assert all(good(o) for o in outs)
    print("handles", len(handles))


def test_next_to_a_capture(problem):
    """Calls on other streams, which obtain memory or take another stream's over, leave a capture under way whole."""
    import torch
    a, b, good, _ = problem
    st = Streams()
    streams = [st.create() for _ in range(34)]
    outs = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in streams]
    cap = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        assert S.call(a, b, cap, stream=torch.cuda.current_stream()) == 0 and not split()
        for s, o in list(zip(streams, outs)) * 2:
            assert S.call(a, b, o, stream=s) == 0
        assert S.call(a, b, cap, stream=torch.cuda.current_stream()) == 0 and not split()
    for _ in range(3):
        cap.zero_()
        graph.replay()
        assert S.call(a, b, outs[0], stream=streams[0]) == 0
        torch.cuda.synchronize()
        assert good(cap) and all(good(o) for o in outs)
    for s in streams:
        st.destroy(s)
