"""The fused bottleneck's forward_steps with a workspace: the pointwise frames
of a chunk as one GEMM, then the depthwise convolution and the pool over them.
Whole-call, uneven and two-frame chunks, and workspaces too small to use,
against the launch per frame bit for bit, with and without updating the state.
"""
import ctypes

import pytest
import torch

from paper_2204_03418_amd import coinf, synth
from parity_util import say
from test_gpu_bneck import BNECK_CASES, DEV, _bneck_parts

pytestmark = pytest.mark.gpu


def _steps(bn, x, cap, frames, update):
    p, w = bn.pool, bn.pw
    z = torch.full((p.batch, p.channels, cap) + p.out_size, float("nan"), dtype=p.torch_dtype,
                   device=DEV)
    frame = w.batch * w.out_channels * w.in_size[0] * w.in_size[1] * x.element_size()
    ws = torch.empty(max(frames * frame, 1), dtype=torch.uint8, device=DEV)
    n = coinf.i32()
    st = coinf.co_bneck_forward_steps_ws(
        bn.handle, ctypes.c_void_p(x.data_ptr()), x.shape[2], ctypes.c_void_p(z.data_ptr()), cap,
        1 if update else 0, ctypes.c_void_p(ws.data_ptr()), frames * frame,
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ctypes.byref(n))
    assert st == coinf.CO_OK
    return z[:, :, :n.value]


@pytest.mark.parametrize("frames", [0, 1, 2, 5, 16])
@pytest.mark.parametrize("case", BNECK_CASES, ids=lambda c: f"bneck_{c[6]}_{c[-1]}_{c[1]}")
def test_bottleneck_chunks(case, frames):
    say("bneck chunks", case, frames)
    B, ci, size, dt, T = case[0], case[1], case[3], case[-1], 16
    xd = synth.normal((B, ci, T) + size, 5600 + ci, dtype=dt).to(DEV)
    _, modules, _, _ = _bneck_parts(case, 5610 + ci)

    def make():
        pw, dw, pool = modules()
        return coinf.Bottleneck(pw, case[8], dw, case[9], pool)

    ref, got = make(), make()
    want = [z for z in (ref.forward_step(xd[:, :, t].contiguous()) for t in range(T))
            if z is not None]
    st = [m.state.clone() for m in (got.pw, got.dw, got.pool)]
    peek = _steps(got, xd, T, frames, False)
    torch.cuda.synchronize()
    assert all(torch.equal(m.state, s) for m, s in zip((got.pw, got.dw, got.pool), st))
    assert (got.pw.steps, got.dw.steps, got.pool.steps) == (0, 0, 0)
    head = _steps(got, xd[:, :, :T - 3].contiguous(), T, frames, True)
    tail = [got.forward_step(xd[:, :, t].contiguous()) for t in range(T - 3, T)]
    outs = [head[:, :, i] for i in range(head.shape[2])] + [z for z in tail if z is not None]
    assert (got.pw.steps, got.dw.steps) == (T, T) and got.pool.steps == ref.pool.steps
    assert len(outs) == len(want) == peek.shape[2]
    for i, w in enumerate(want):
        assert torch.equal(outs[i], w) and torch.equal(peek[:, :, i], w)


@pytest.mark.parametrize("case", BNECK_CASES, ids=lambda c: f"bneck_{c[6]}_{c[-1]}_{c[1]}")
def test_bottleneck_workspace_bytes(case):
    """The chunk tests above have layers that the two launches take, and the
    library asks for a workspace from three frames on (of a small layer)."""
    _, modules, _, _ = _bneck_parts(case, 5690)
    pw, dw, pool = modules()
    bn = coinf.Bottleneck(pw, case[8], dw, case[9], pool)
    nb = coinf.i64()

    def frames(T):
        assert coinf.co_bneck_workspace_bytes(bn.handle, T, ctypes.byref(nb)) == coinf.CO_OK
        return nb.value // (pw.batch * pw.out_channels * pw.in_size[0] * pw.in_size[1] *
                            (2 if case[-1] == "bf16" else 4))

    assert [frames(T) for T in (0, 1, 2, 3, 16)] == [0, 0, 0, 3, 16]


def test_bottleneck_workspace_past_the_launches():
    """A workspace that holds more frames than one launch addresses (2 GiB of
    pointwise frames) is used in chunks that a launch takes."""
    B, ci, co, size, T = 64, 16, 432, (7, 7), 900
    say("bneck large workspace")
    x = synth.normal((B, ci, T) + size, 5700, dtype="bf16").to(DEV)
    w1 = synth.normal((co, ci, 1, 1, 1), 5701, dtype="bf16")
    w2 = synth.normal((co, 1, 3, 3, 3), 5702, dtype="bf16") * 0.2

    def make():
        pool = coinf.CoPool("avg", batch=B, channels=co, kernel=(4,) + size, in_size=size,
                            stride=(1,) + size, dtype=torch.bfloat16)
        pw = coinf.CoConv(w1.to(DEV), batch=B, in_size=size)
        dw = coinf.CoConv(w2.to(DEV), batch=B, in_size=size, groups=co, padding=(0, 1, 1))
        return coinf.Bottleneck(pw, True, dw, True, pool)

    frame = B * co * 49 * 2
    ws = torch.zeros(T * frame, dtype=torch.uint8, device=DEV)
    assert ws.numel() > 2 ** 31
    outs = []
    for space in (ws, None):
        bn = make()
        z = torch.empty((B, co, T, 1, 1), dtype=torch.bfloat16, device=DEV)
        n = coinf.i32()
        assert coinf.co_bneck_forward_steps_ws(
            bn.handle, x.data_ptr(), T, z.data_ptr(), T, 1,
            None if space is None else space.data_ptr(), 0 if space is None else space.numel(),
            torch.cuda.current_stream().cuda_stream, ctypes.byref(n)) == coinf.CO_OK
        outs.append(z[:, :, :n.value])
    assert bool(ws[:frame].any())
    assert outs[0].shape[2] > 0 and torch.equal(*outs)
