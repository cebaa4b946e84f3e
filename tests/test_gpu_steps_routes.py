"""forward_steps on each persistent kernel at the calls that it is chosen for,
time segments among them: bit for bit the outputs of single steps, whole, as
the continuation of single steps, before them, and without updating the state.
The route is asserted, so that a change of the choice cannot leave a kernel
untested.
"""
import pytest
import torch

from paper_2204_03418_amd import coinf, synth
from parity_util import say

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")

CASES = [
    # route, dtype, B, Cin, Cout, kernel, size, stride, padding, dilation, T
    # register GEMM, one spatial tap: every instantiation, segments (T >= 8 (kT - 1))
    ("reg", "f32", 4, 64, 64, (3, 1), (25,), (1, 1), (1, 0), (1, 1), 4),
    ("reg", "f32", 32, 64, 256, (9, 1), (25,), (1, 1), (4, 0), (1, 1), 16),
    ("reg", "f32", 1, 128, 128, (3, 1), (25,), (1, 1), (0, 0), (1, 1), 64),      # segments
    ("reg", "f32", 3, 100, 72, (3, 1), (11,), (1, 1), (2, 0), (1, 1), 50),       # ragged, segments
    ("reg", "bf16", 64, 64, 256, (3, 1), (25,), (1, 1), (0, 0), (1, 1), 5),
    ("reg", "bf16", 32, 64, 256, (9, 1), (25,), (1, 1), (4, 0), (1, 1), 64),     # segments
    ("reg", "bf16", 64, 128, 128, (3, 1), (25,), (1, 1), (1, 0), (1, 1), 16),
    ("reg", "bf16", 32, 128, 128, (9, 1), (25,), (1, 1), (0, 0), (1, 1), 17),
    # with temporal stride and dilation: step plans, segments
    ("reg", "f32", 1, 128, 128, (3, 1), (25,), (2, 1), (0, 0), (1, 1), 65),
    ("reg", "f32", 2, 128, 128, (2, 1), (11,), (2, 1), (0, 0), (1, 1), 100),
    ("reg", "f32", 2, 128, 128, (3, 1), (25,), (1, 1), (1, 0), (2, 1), 150),
    ("reg", "f32", 32, 64, 256, (9, 1), (25,), (2, 1), (4, 0), (1, 1), 16),
    ("reg", "bf16", 32, 64, 256, (9, 1), (25,), (2, 1), (4, 0), (1, 1), 9),
    ("reg", "bf16", 64, 128, 128, (3, 1), (25,), (2, 1), (1, 0), (1, 1), 9),
    ("reg", "bf16", 32, 128, 128, (9, 1), (25,), (2, 1), (0, 0), (1, 1), 11),
    # persistent 3x3 GEMM: pixel pairs and single pixels, kT 2, ragged channels
    ("gemm", "bf16", 64, 96, 96, (3, 3, 3), (14, 14), (1, 1, 1), (1, 1, 1), (1, 1, 1), 9),
    ("gemm", "bf16", 64, 72, 80, (2, 3, 3), (14, 10), (1, 1, 1), (0, 1, 1), (1, 1, 1), 4),
    ("gemm", "bf16", 16, 192, 192, (3, 3, 3), (14, 14), (1, 1, 1), (0, 1, 1), (1, 1, 1), 9),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "_".join(map(str, c[:6])) + f"_s{c[7][0]}_T{c[10]}")
def test_persistent_route(case):
    route, dt, B, cin, cout, k, size, st, p, dil, T = case
    say("route", case)
    g = torch.Generator(device=DEV).manual_seed(98700 + cin + T)
    tdt = synth.torch_dtype(dt)
    x = torch.randn((B, cin, T + 5) + size, generator=g, device=DEV).to(tdt)
    w = (torch.randn((cout, cin) + k, generator=g, device=DEV) * 0.05).to(tdt)
    b = torch.randn((cout,), generator=g, device=DEV).to(tdt)

    def make():
        return coinf.CoConv(w, b, batch=B, in_size=size, stride=st, padding=p, dilation=dil)

    a, c = make(), make()
    assert a.steps_route(T) == route
    seq = [c.forward_step(x[:, :, t].contiguous()) for t in range(T + 5)]

    def frames(lo, hi):
        f = [s for s in seq[lo:hi] if s is not None]
        return torch.stack(f, 2) if f else None

    def same(got, want):
        return (got is None and want is None) or torch.equal(got, want)

    assert same(a.forward_steps(x[:, :, :T].contiguous()), frames(0, T))
    assert all(same(a.forward_step(x[:, :, t].contiguous()), seq[t]) for t in range(T, T + 5))
    d = make()
    for t in range(3):
        d.forward_step(x[:, :, t].contiguous())
    before = d.state.clone()
    part = x[:, :, 3:T + 3].contiguous()
    assert same(d.forward_steps(part, update_state=False), frames(3, T + 3))
    assert d.steps == 3 and torch.equal(d.state, before)
    assert same(d.forward_steps(part), frames(3, T + 3))
    assert all(same(d.forward_step(x[:, :, t].contiguous()), seq[t]) for t in range(T + 3, T + 5))


@pytest.mark.parametrize("update", [True, False], ids=["update", "peek"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_loop_in_a_graph(dt, update):
    """A call that runs as single steps, recorded into a graph: one that would
    allocate (the ring's backup, copies of frames at odd strides) takes a launch
    that needs no memory instead.  Every replay, with eager work in between,
    gives the outputs and the state of the eager call from the same state."""
    B, C, T = 4, 192, 3
    say("loop in a graph", dt, update)
    g = torch.Generator(device=DEV).manual_seed(98800 + update)
    tdt = synth.torch_dtype(dt)
    x = torch.randn((B, C, T + 2, 7, 7), generator=g, device=DEV).to(tdt)
    w = (torch.randn((C, C, 3, 3, 3), generator=g, device=DEV) * 0.05).to(tdt)
    eager, co = (coinf.CoConv(w, None, batch=B, in_size=(7, 7), padding=(0, 1, 1))
                 for _ in range(2))
    assert co.steps_route(T, update_state=update) == "loop"
    for t in range(2):
        eager.forward_step(x[:, :, t].contiguous())
        co.forward_step(x[:, :, t].contiguous())
    buf, start = x[:, :, 2:].contiguous(), eager.state.clone()
    want = eager.forward_steps(buf, update_state=update)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = co.forward_steps(buf, update_state=update)
    for _ in range(3):
        co.state.copy_(start)
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.equal(co.state, eager.state)
        assert torch.isfinite(buf.float().sum())
