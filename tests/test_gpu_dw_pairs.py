"""Depthwise forward_steps with two outputs of a row per thread (planes of
more than 64 pixels): odd and even widths, no padding to more than a stencil's
reach, row strides and dilations, both stencils, every kT, and a two-column
plane.  Each against the oracle and bit for bit against single steps, as a
clip, as the continuation of single steps, before them, and without updating
the state.
"""
import pytest

from paper_2204_03418_amd import coinf, synth
from parity_util import oracle_conv, say
from test_gpu_parity import DEV, _check_fused_steps

pytestmark = pytest.mark.gpu

CASES = [
    # B, C, kernel, size, stride, padding, dilation
    (2, 5, (3, 3, 3), (13, 12), (1, 1, 1), (0, 1, 1), (1, 1, 1)),
    (3, 4, (2, 3, 3), (9, 11), (1, 1, 1), (1, 0, 0), (1, 1, 1)),
    (2, 3, (4, 3, 3), (10, 9), (1, 2, 1), (2, 2, 2), (1, 1, 1)),
    (1, 6, (5, 3, 3), (17, 8), (1, 1, 1), (4, 1, 3), (1, 2, 1)),
    (2, 3, (1, 3, 3), (40, 2), (1, 1, 1), (0, 1, 1), (1, 1, 1)),
    (2, 7, (5, 1, 1), (9, 15), (1, 1, 1), (0, 0, 0), (1, 1, 1)),
    (2, 3, (3, 1, 1), (8, 10), (1, 1, 1), (1, 0, 1), (1, 1, 1)),
]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "_".join(map(str, c[2] + c[3])))
def test_depthwise_pairs(case, dt):
    B, C, k, size, st, p, dil = case
    say("dw pairs", case, dt)
    spec = synth.ConvSpec(batch=B, in_channels=C, out_channels=C, kernel=k, in_size=size,
                          stride=st, padding=p, dilation=dil, groups=C, dtype=dt)
    x, w, b = synth.conv_inputs(spec, 14, 99500 + 7 * C + k[0], "kaiming")

    def make():
        return coinf.CoConv(w.to(DEV), b.to(DEV), batch=B, in_size=size, stride=st, padding=p,
                            dilation=dil, groups=C, algo="depthwise")

    _check_fused_steps(make, x, oracle_conv(w, b, st, p, dil, C), synth.torch_dtype(dt),
                       "dw pairs")
