"""Global pools on the frames-in-lanes kernel: buffers of frames and clips.

At the edges of its range: windows of 1 to 64 frames (every size of the
temporal tree), planes of 1 to 64 pixels, calls of less than, exactly and
more than a block of 64 frames, dilated windows up to the longest history,
averages over the real frames only, and clips whose last 16 bytes are not a
whole unit.  Each against the oracle and bit for bit against single steps.
"""
import pytest
import torch

import oracle
from paper_2204_03418_amd import coinf, synth
from parity_util import assert_close, np64, say, window_terms

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")

CASES = [
    # kind, B, C, T, kT, (H, W), sT, pT, dT, count_include_pad, dtype
    ("avg", 2, 5, 70, 64, (7, 7), 1, 0, 1, True, "f32"),     # widest window, two blocks
    ("avg", 1, 3, 64, 33, (8, 8), 1, 16, 1, False, "bf16"),  # real frames only, padded ends
    ("max", 3, 7, 65, 17, (5, 7), 2, 8, 3, True, "bf16"),    # dilated, strided, one frame over
    ("max", 1, 2, 140, 64, (3, 3), 1, 32, 2, True, "f32"),   # span 127, three blocks
    ("avg", 2, 9, 9, 9, (4, 4), 3, 2, 1, False, "f32"),      # a call as long as the window
    ("avg", 1, 33, 20, 16, (1, 1), 1, 0, 1, True, "bf16"),   # one pixel a plane
    ("max", 2, 130, 7, 2, (6, 5), 1, 1, 1, True, "bf16"),    # short call, ragged planes
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "_".join(map(str, c[:5])))
def test_frames_in_lanes_pool(case):
    kind, B, C, T, kT, size, sT, pT, dT, cip, dt = case
    say("pool frames", case)
    tdt = synth.torch_dtype(dt)
    k, st, p, d = (kT,) + size, (sT,) + size, (pT, 0, 0), (dT, 1, 1)
    x = synth.normal((B, C, T) + size, 5200 + 7 * kT + C, dtype=dt)
    xd = x.to(DEV)

    def make():
        return coinf.CoPool(kind, batch=B, channels=C, kernel=k, in_size=size, stride=st,
                            padding=p, dilation=d, count_include_pad=cip, dtype=tdt)

    po, ref = make(), oracle.ContinualPool(kind, k, st, p, d, cip, spatial_dims=2)
    assert po.steps_fused(T, pad_end=True)
    want = ref.forward_steps(np64(x), pad_end=True)
    got = po.forward_steps(xd, pad_end=True)
    assert_close(np64(got), want, tdt, "frames pool steps", terms=window_terms(k))
    # a clip is a stream that begins and ends with it
    assert torch.equal(make().forward(xd), got)
    # single steps, a buffer that continues them, and single steps after it
    a, b = make(), make()
    seq = [b.forward_step(xd[:, :, t].contiguous()) for t in range(T)]
    cut, end = 3, max(4, T - 2)
    parts = [a.forward_step(xd[:, :, t].contiguous()) for t in range(cut)]
    n, before = a.steps, a.state.clone()
    peek = a.forward_steps(xd[:, :, cut:end].contiguous(), update_state=False)
    assert a.steps == n and torch.equal(a.state, before)
    mid = a.forward_steps(xd[:, :, cut:end].contiguous())
    assert (mid is None and peek is None) or torch.equal(mid, peek)
    parts += [] if mid is None else [mid[:, :, i] for i in range(mid.shape[2])]
    parts += [a.forward_step(xd[:, :, t].contiguous()) for t in range(end, T)]
    parts, seq = [q for q in parts if q is not None], [q for q in seq if q is not None]
    assert len(parts) == len(seq)
    for g_, s_ in zip(parts, seq):
        assert torch.equal(g_, s_)


FORMS = [
    # short calls of many planes: several planes in a pass, ragged last ones
    ("avg", 8, 2050, 8, 4, (2, 2), 1, 0, 1, True, "f32"),
    ("max", 4, 4100, 9, 3, (1, 3), 2, 1, 2, True, "bf16"),
    ("avg", 2, 8200, 8, 4, (4, 4), 1, 1, 1, False, "bf16"),
    ("avg", 1, 16500, 21, 9, (5, 5), 1, 4, 1, False, "f32"),
    # long clips of few planes: segments of the time axis, with and without
    # blocks before them that their windows reach back to
    ("max", 1, 3, 1500, 64, (3, 3), 1, 32, 2, True, "f32"),
    ("avg", 1, 2, 1300, 40, (4, 4), 1, 20, 1, False, "bf16"),
    ("max", 1, 2, 700, 5, (7, 7), 3, 2, 1, True, "bf16"),
    ("avg", 1, 1, 900, 1, (1, 1), 1, 0, 1, True, "f32"),
]


@pytest.mark.parametrize("case", FORMS, ids=lambda c: "_".join(map(str, c[:5])))
def test_frames_in_lanes_pool_forms(case):
    test_frames_in_lanes_pool(case)
