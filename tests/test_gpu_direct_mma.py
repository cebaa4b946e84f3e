"""Direct layers on the matrix cores, at the edges of their tiles and forms:
channel counts and depths that fill no tile, fragment or k-step, spatial and
temporal strides and dilations, even kernels, planes smaller than a tile,
rows of one pixel, both pixel tiles and every channel tile, both dtypes.
Each against the oracle and bit for bit against single steps, as a clip, as
the continuation of single steps, before them, and without updating the state.
"""
import ctypes

import pytest
import torch

from paper_2204_03418_amd import coinf, synth
from parity_util import assert_close, conv_terms, np64, oracle_conv, say
from test_gpu_parity import DEV, _check_fused_steps

pytestmark = pytest.mark.gpu

CASES = [
    # B, Cin, Cout, kernel, size, stride, padding, dilation, dtype, T, algo
    (3, 24, 48, (3, 3, 3), (15, 14), (1, 2, 2), (1, 1, 1), (1, 1, 1), "bf16", 14, "direct"),
    (2, 29, 97, (3, 3, 3), (9, 17), (1, 2, 2), (2, 1, 1), (1, 1, 1), "f32", 13, "direct"),
    (2, 96, 192, (3, 3, 3), (11, 11), (1, 2, 2), (1, 1, 1), (1, 1, 1), "bf16", 13, "auto"),
    (1, 80, 130, (2, 3, 3), (10, 7), (2, 2, 1), (1, 0, 1), (1, 1, 1), "bf16", 15, "direct"),
    (2, 40, 64, (3, 2, 4), (13, 12), (1, 3, 2), (2, 1, 2), (2, 1, 1), "f32", 16, "direct"),
    (2, 17, 33, (4, 3, 3), (12, 9), (3, 1, 1), (4, 2, 0), (2, 2, 1), "bf16", 18, "direct"),
    (5, 70, 80, (5, 5), (31,), (1, 2), (2, 2), (1, 1), "bf16", 20, "direct"),
    (17, 64, 40, (3,), (), (1,), (0,), (1,), "f32", 30, "direct"),          # one pixel a frame
    (4, 100, 70, (5,), (), (2,), (3,), (3,), "bf16", 40, "direct"),
    (2, 33, 128, (1, 3, 3), (16, 16), (1, 2, 2), (0, 1, 1), (1, 1, 1), "f32", 12, "direct"),
    (16, 40, 128, (3, 3, 3), (20, 20), (1, 1, 1), (1, 1, 1), (1, 1, 1), "bf16", 12, "direct"),
    (2, 5, 64, (3, 3, 3), (24, 24), (1, 1, 1), (0, 1, 1), (1, 1, 1), "f32", 12, "direct"),
    (16, 24, 64, (2, 3, 3), (33, 29), (1, 2, 2), (1, 1, 1), (1, 1, 1), "f32", 24, "direct"),
]


def _id(c):
    return "_".join(map(str, c[:4])) + c[8]


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_direct_mma_steps(case):
    B, cin, cout, k, size, st, p, dil, dt, T, algo = case
    say("direct mma", case)
    spec = synth.ConvSpec(batch=B, in_channels=cin, out_channels=cout, kernel=k, in_size=size,
                          stride=st, padding=p, dilation=dil, dtype=dt)
    x, w, b = synth.conv_inputs(spec, T, 99100 + 7 * cin + cout, "kaiming")

    def make():
        return coinf.CoConv(w.to(DEV), b.to(DEV), batch=B, in_size=size, stride=st, padding=p,
                            dilation=dil, algo=algo)

    assert make().algo == "direct"
    _check_fused_steps(make, x, oracle_conv(w, b, st, p, dil, 1), synth.torch_dtype(dt),
                       "direct mma")


@pytest.mark.parametrize("scaled", [False, True])
def test_direct_mma_infinite_frames(scaled):
    """Infinities and NaN in bf16 frames reach the outputs their taps feed and
    no others, with plain and with folded (float32) weights; the clip equals
    forward_steps with end padding."""
    say("direct mma inf", scaled)
    spec = synth.ConvSpec(batch=2, in_channels=24, out_channels=48, kernel=(3, 3, 3),
                          in_size=(9, 8), stride=(1, 2, 2), padding=(1, 1, 1), dtype="bf16")
    x, w, b = synth.conv_inputs(spec, 6, 99300, "kaiming")
    x[0, 3, 2, 4, 4] = float("inf")
    x[1, 5, 1, 2, 6] = float("-inf")
    x[1, 7, 4, 0, 0] = float("nan")
    bn = None
    if scaled:
        bn = (synth.normal((48,), 99310).abs() + 0.5, synth.normal((48,), 99311),
              synth.normal((48,), 99312), synth.normal((48,), 99313).abs() + 0.5, 1e-5)
        bn = tuple(t.to(DEV) if torch.is_tensor(t) else t for t in bn)

    def make():
        return coinf.CoConv(w.to(DEV), b.to(DEV), batch=2, in_size=(9, 8), stride=(1, 2, 2),
                            padding=(1, 1, 1), algo="direct", bn=bn)

    got = make().forward(x.to(DEV))
    assert torch.equal(got.nan_to_num(7e7, 8e7, -8e7),
                       make().forward_steps(x.to(DEV), pad_end=True).nan_to_num(7e7, 8e7, -8e7))
    w64, b64 = w.double(), b.double()
    if scaled:
        g, be, mu, var, eps = [t.cpu().double() if torch.is_tensor(t) else t for t in bn]
        sc = g / (var + eps).sqrt()
        w64, b64 = w64 * sc.view(-1, 1, 1, 1, 1), b64 * sc + be - mu * sc
    want = torch.nn.functional.conv3d(x.double(), w64, b64, (1, 2, 2), (1, 1, 1))
    got = got.cpu().double()
    for kind in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(kind(got), kind(want))
    ok = torch.isfinite(want)
    assert_close(np64(got[ok]), np64(want[ok]), torch.bfloat16, "direct mma inf",
                 terms=conv_terms(w))


@pytest.mark.parametrize("marked", [True, False])
def test_direct_mma_attached_state(marked):
    """A state attached mid-stream continues bit for bit; one whose header
    does not say what its weights are (as earlier versions wrote them) takes
    the float32 instructions and stays within the bound."""
    say("direct mma attach", marked)
    spec = synth.ConvSpec(batch=2, in_channels=40, out_channels=64, kernel=(3, 3, 3),
                          in_size=(9, 8), stride=(1, 2, 2), padding=(0, 1, 1), dtype="bf16")
    x, w, b = synth.conv_inputs(spec, 8, 99400, "kaiming")
    xd, wd, bd = x.to(DEV), w.to(DEV), b.to(DEV)
    kw = dict(batch=2, in_size=(9, 8), stride=(1, 2, 2), padding=(0, 1, 1), algo="direct")
    a = coinf.CoConv(wd, bd, **kw)
    a.forward_steps(xd[:, :, :3].contiguous())
    state = a.state.clone()
    if not marked:
        state[32:256] = 0
    c = coinf.CoConv(wd, bd, state=state, attach_steps=3, **kw)
    want = a.forward_steps(xd[:, :, 3:].contiguous())
    got = c.forward_steps(xd[:, :, 3:].contiguous())
    if marked:
        assert torch.equal(got, want)
    ref = torch.nn.functional.conv3d(x.double(), w.double(), b.double(), (1, 2, 2), (0, 1, 1))
    assert_close(np64(got), np64(ref[:, :, 1:]), torch.bfloat16, "attached",
                 terms=conv_terms(w))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_direct_mma_buffer_past_32_bits(dt):
    """A buffer whose planes lie past 32-bit offsets steps frame by frame, with
    the bits of steps on single frames."""
    T, hw = (15 if dt == "f32" else 29), 1024
    say("direct mma large buffer", dt)
    g = torch.Generator(device=DEV).manual_seed(99500)
    x = torch.randn((1, 32, T, hw, hw), generator=g, device=DEV).to(synth.torch_dtype(dt))
    assert 32 * T * hw * hw * x.element_size() >= 0x70000000
    w = synth.normal((16, 32, 2, 3, 3), 99501, dtype=dt, std=0.1).to(DEV)
    a, c = (coinf.CoConv(w, batch=1, in_size=(hw, hw), stride=(1, 2, 2), padding=(0, 1, 1),
                         algo="direct") for _ in range(2))
    assert not a.steps_fused(T) and a.steps_fused(2)
    got = a.forward_steps(x)
    steps = [c.forward_step(x[:, :, t].contiguous()) for t in range(T)]
    assert torch.equal(got, torch.stack([s for s in steps if s is not None], 2))


@pytest.mark.parametrize("scaled", [False, True])
def test_direct_mma_output_past_32_bits(scaled):
    """The same of output planes: a small call into a large output buffer."""
    B, T, cap = 2, 5, 3700000
    say("direct mma large output", scaled)
    x = synth.normal((B, 32, T, 7, 8), 99510, dtype="bf16").to(DEV)
    w = synth.normal((20, 32, 2, 3, 3), 99511, dtype="bf16", std=0.1).to(DEV)
    bn = tuple(synth.normal((20,), 99512 + i).abs().to(DEV) + 0.5 for i in range(4)) + (1e-5,)
    a, c = (coinf.CoConv(w, batch=B, in_size=(7, 8), stride=(1, 2, 2), padding=(0, 1, 1),
                         algo="direct", bn=bn if scaled else None) for _ in range(2))
    assert 20 * cap * 16 * 2 >= 0x70000000
    y = torch.zeros((B, 20, cap, 4, 4), dtype=torch.bfloat16, device=DEV)
    n = coinf.i32()
    assert coinf.co_conv_forward_steps(a.handle, x.data_ptr(), T, y.data_ptr(), cap, 0, 1,
                                       torch.cuda.current_stream().cuda_stream,
                                       ctypes.byref(n)) == coinf.CO_OK
    steps = [c.forward_step(x[:, :, t].contiguous()) for t in range(T)]
    want = torch.stack([s for s in steps if s is not None], 2)
    assert n.value == want.shape[2] and torch.equal(y[:, :, :n.value], want)
    assert not bool(y[:, :, n.value:n.value + 4].any()) and not bool(y[:, :, -1].any())
