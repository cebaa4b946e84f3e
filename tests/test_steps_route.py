"""Which way forward_steps takes (host only).

The layers and calls below were measured every way they can run (the GEMM over
frames, a persistent launch, single steps): the route is one within a tenth of
the fastest.  And the tests of a kernel reach that kernel.
"""
import ctypes

import pytest

import test_gpu_clip_gemm
import test_gpu_direct_mma
from paper_2204_03418_amd import coinf as C

SKELETON = dict(kernel=(9, 1), in_size=(25,))


def route(T, dt, batch, cin, cout, kernel, in_size=(), stride=1, padding=0, dilation=1,
          algo="auto", update=True, cap=None):
    d = C.conv_desc(batch, cin, cout, kernel, in_size, stride, padding, dilation,
                    dtype=C.CO_F32 if dt == "f32" else C.CO_BF16, algo=algo)
    return C.conv_steps_route(d, T, T if cap is None else cap, update)


def video(hw):
    return dict(kernel=(3, 3, 3), in_size=(hw, hw), padding=(0, 1, 1))


MEASURED = [
    # microseconds: GEMM over frames / persistent / single steps
    ("f32", 64, 128, 128, dict(kernel=(3, 1), in_size=(25,)), 2, ("loop", "reg")),    # 51/18/15
    ("f32", 64, 128, 128, dict(kernel=(3, 1), in_size=(25,)), 8, ("reg",)),           # 61/29/61
    ("f32", 32, 128, 128, dict(kernel=(3, 1), in_size=(25,)), 300, ("clip",)),        # 220/279/-
    ("f32", 32, 64, 256, SKELETON, 4, ("loop", "reg")),                               # 81/34/34
    ("f32", 32, 64, 256, SKELETON, 16, ("reg",)),                                     # 97/55/138
    ("f32", 16, 128, 128, SKELETON, 4, ("loop",)),                                    # 132/-/25
    ("f32", 16, 128, 128, SKELETON, 150, ("clip",)),                                  # 228/-/840
    ("bf16", 64, 128, 128, dict(kernel=(3, 1), in_size=(25,)), 8, ("reg",)),          # 25/12/46
    ("bf16", 32, 128, 128, SKELETON, 8, ("reg",)),                                    # 51/19/51
    ("bf16", 16, 64, 256, SKELETON, 8, ("reg",)),                                     # 38/19/49
    ("bf16", 32, 64, 256, SKELETON, 300, ("reg",)),  # 142/149/- (129/97 with repeated frames)
    ("bf16", 16, 64, 256, SKELETON, 300, ("clip",)),                                  # 67/111/-
    ("bf16", 64, 64, 64, SKELETON, 300, ("clip",)),                                   # 81/111/-
    ("f32", 64, 64, 256, SKELETON, 8, ("reg",)),                                      # 93/64/105
    ("bf16", 64, 128, 128, dict(kernel=(3, 1), in_size=(25,)), 300, ("clip",)),       # 104/253/-
    ("f32", 1, 128, 128, dict(kernel=(3, 1), in_size=(25,), stride=(2, 1)), 8, ("reg",)),  # 57/16/40
    ("f32", 1, 128, 128, dict(kernel=(3, 1), in_size=(25,), stride=(2, 1)), 300, ("reg",)),  # 57/35/-
    ("bf16", 32, 64, 256, dict(SKELETON, stride=(2, 1)), 8, ("reg",)),                # 39/15/50
    ("bf16", 32, 64, 256, dict(SKELETON, stride=(2, 1)), 150, ("clip",)),             # 57/102/-
    ("f32", 4, 192, 192, video(7), 4, ("loop",)),                                     # 543/-/139
    ("f32", 4, 192, 192, video(7), 64, ("clip",)),                                    # 557/-/2539
    ("f32", 1, 192, 192, video(7), 16, ("clip",)),                                    # 545/-/917
    ("f32", 1, 96, 96, dict(kernel=(1, 3, 3), in_size=(14, 14), padding=(0, 1, 1)), 2, ("loop",)),
    ("f32", 1, 96, 96, dict(kernel=(1, 3, 3), in_size=(14, 14), padding=(0, 1, 1)), 16, ("clip",)),
    ("bf16", 1, 64, 128, video(7), 4, ("loop",)),                                     # 65/-/21
    ("bf16", 64, 192, 192, video(14), 16, ("gemm",)),                                 # 688/358/-
    ("bf16", 4, 96, 96, video(14), 64, ("clip",)),                                    # 118/575/1086
    ("bf16", 16, 192, 432, dict(kernel=(1, 1, 1), in_size=(7, 7)), 2, ("clip",)),     # 10/-/14
    ("bf16", 16, 192, 432, dict(kernel=(1, 1, 1), in_size=(7, 7)), 64, ("clip",)),    # 31/-/455
    ("f32", 16, 24, 108, dict(kernel=(1, 1, 1), in_size=(14, 14)), 64, ("clip",)),    # 36/-/321
]


@pytest.mark.parametrize("case", MEASURED, ids=lambda c: "_".join(map(str, c[:4])) + f"_T{c[5]}")
def test_route_of_measured_calls(case):
    dt, B, cin, cout, layer, T, want = case
    assert route(T, dt, B, cin, cout, **layer) in want


def test_peek_prefers_one_launch():
    """Without updating the state the GEMM has no second pass, and a loop has
    the ring's backup to pay."""
    layer = dict(dt="bf16", batch=64, cin=64, cout=64, **SKELETON)
    assert route(2, **layer) in ("loop", "reg")          # 12 and 18 against 27
    assert route(2, update=False, **layer) == "clip"     # 9.9 against 18 and 44


def test_route_arguments():
    d = C.conv_desc(1, 2, 3, (3,), ())
    r = C.i32()
    assert C.co_conv_steps_route(ctypes.byref(d), -1, 0, 1, ctypes.byref(r)) == C.CO_EINVAL
    assert C.co_conv_steps_route(ctypes.byref(d), 1, -1, 1, ctypes.byref(r)) == C.CO_EINVAL
    assert C.co_conv_steps_route(ctypes.byref(d), 1, 1, 1, None) == C.CO_EINVAL
    d.groups = 7
    assert C.co_conv_steps_route(ctypes.byref(d), 1, 1, 1, ctypes.byref(r)) == C.CO_EINVAL


@pytest.mark.parametrize("case", test_gpu_clip_gemm.CASES, ids=lambda c: "_".join(map(str, c[:4])))
def test_clip_gemm_tests_reach_it(case):
    B, cin, cout, k, size, st, p, dil, dt, T, algo = case
    layer = dict(kernel=k, in_size=size, stride=st, padding=p, dilation=dil, algo=algo)
    assert route(T, dt, B, cin, cout, **layer) == "clip"


@pytest.mark.parametrize("case", test_gpu_direct_mma.CASES, ids=lambda c: "_".join(map(str, c[:4])))
def test_direct_mma_tests_reach_it(case):
    B, cin, cout, k, size, st, p, dil, dt, T, algo = case
    layer = dict(kernel=k, in_size=size, stride=st, padding=p, dilation=dil, algo=algo)
    assert route(T, dt, B, cin, cout, **layer) == "direct_mma"
