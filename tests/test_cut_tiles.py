"""1-byte outputs of a token tile that the end of the tokens cuts: every number of tokens left of its last 16, in the kernels
that stage them, in both orders, with Sum (whose operand may not be read past the end) and a table.  Exact; what is past
the end stays untouched."""
import os
import sys

import numpy as np
import pytest

import oracle
import workloads as wl

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "emu"))
import build_emu  # noqa: E402
from test_emulated_kernels import run_case  # noqa: E402

TUNINGS = [(128, 16), (96, 16), (128, 8), (128, 112), (128, 108), (96, 112), (64, 112), (128, 132), (96, 132), (64, 132), (64, 134), (32, 134)]


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("M,out_type,postop,tm,variant,extra", [
    (129, "s8", "gelu", 128, 16, {}), (191, "u8", "none", 96, 16, {"xtiled": "out"}), (143, "s8", "none", 128, 112, {"ldo": 149}),
    (70, "s8", "gelu", 64, 112, {"xtiled": "out"}), (107, "u8", "gelu", 128, 108, {}), (125, "s8", "none", 96, 132, {})])
def test_cut_tiles_on_the_cpu(M, out_type, postop, tm, variant, extra):
    build_emu.build()
    res = run_case(200, 600, M, 0.9, out_type, postop, tm, variant, cus=2, **extra)
    assert res["match"] and res["padding_untouched"], res


@pytest.mark.gpu
@pytest.mark.parametrize("left", range(1, 16))
def test_cut_tiles_on_the_device(left):
    from test_gpu_parity import _run_sum, _run_tiled_out, assert_parity, check_case, oracle_spmm
    for i, tuning in enumerate(TUNINGS):
        M = (64, 128, 160, 32)[(i + left) % 4] + left
        case = wl.Case("cut", 200, 600, M, (0.9, 0.8)[left % 2], wl.N4K1, ("s8", "u8")[i % 2], "gelu", keys=(110, M, i))
        check_case(case, tuning=tuning, ldo=M + (16 - left, 0, 5)[i % 3])
        d = wl.make(case)
        assert_parity(_run_tiled_out(d, case, tuning, i % 2 == 0), oracle_spmm(d["W"], d["X"], d, case), case)
        case = case.with_(postop="none")
        d = wl.make(case)
        R = (wl.rng_for(111, 200, M).standard_normal((200, M)) * wl.preact_sigma(600, case.sparsity)).astype(np.float32)
        ref = oracle.spmm(d["W"], d["X"], d["w_scale"], d["x_scale"], d["bias"], "none", case.out_type, d["out_scale"], d["out_zero_point"],
                          d["mid_scale"], d["x_zero_point"], sum=R)
        assert_parity(_run_sum(d, case, R, M, tuning, 0), ref, case)
