"""Short batches whose workgroups are dealt to the XCDs in equal parts, where slices of the row groups and of the tokens would give
some XCD a round of workgroups more: every number is dealt once, in both orders, by both bodies of the short-batch kernels, and the
measured times bear the rule out."""
import csv
import os
import sys

import numpy as np
import pytest

import paper_2306_16601_amd as sp
import workloads as wl

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "emu"))
import build_emu  # noqa: E402
from test_emulated_kernels import run_case  # noqa: E402


# (N, K, M, tuning, workgroups): 33 to 42 of an XCD's 32 CUs by slices
PROBLEMS = [
    (768, 3072, 333, None, 256),            # 12 x 21, 4 row tiles to a workgroup
    (1300, 650, 665, (32, 101), 232),       # 11 x 21
    (2304, 2304, 400, (32, 104), 240),      # 18 x 13, ring
    (1300, 2600, 346, (16, 103), 248),      # 11 x 22
    (640, 1100, 380, (16, 106), 240),       # 10 x 24
    (2304, 4096, 797, (64, 104), 240),      # 18 x 13
]


@pytest.mark.parametrize("N,K,M,tuning,workgroups", PROBLEMS)
def test_one_round_of_workgroups(N, K, M, tuning, workgroups):
    W = np.zeros((N, K), dtype=np.int8)
    W[::4, ::5] = 1
    h = sp.spmm_pack_host(W)
    try:
        if tuning:
            sp.spmm_set_tuning(h, *tuning)
        here = sp.spmm_plan(h, M, "f32")
        assert here[2] == workgroups <= 256, here
        assert -(-N // here[1]) * -(-M // here[0]) <= workgroups
    finally:
        sp.spmm_destroy(h)


@pytest.mark.parametrize("us", ["us", "graph"])        # launches back to back, and replayed from a graph
def test_dealing_gains_wherever_it_saves_a_round(us):
    """What a comment in spmm_plan.hip says of profiles/spmm_plan_equal_parts.csv."""
    table = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles", "spmm_plan_equal_parts.csv")
    rows = list(csv.DictReader(line for line in open(table) if not line.startswith("#")))

    def ratios(which):
        return np.array([float(r[us + "_equal"]) / float(r[us + "_slices"]) for r in rows if which(r)])

    def one_segment(r):
        return int(r["problem"].split()[0].split("x")[1]) <= 512

    forced, two = ratios(lambda r: r["configuration"] != "auto"), [r for r in rows if r["rounds_slices"] == "2"]
    assert len(forced) >= 100 and forced.max() < 1
    for ring, alone, most in ((False, False, 0.77), (False, True, 0.90), (True, False, 0.67)):
        of = ratios(lambda r: r in two and r["configuration"].endswith("/104") == ring and (one_segment(r) or not alone))
        assert len(of) >= 8 and np.exp(np.log(of).mean()) <= most
    automatic = ratios(lambda r: r["configuration"] == "auto")
    assert len(automatic) >= 60 and np.exp(np.log(automatic).mean()) <= 0.965
    assert (automatic > 1.03).sum() <= 2 and automatic.max() <= 1.09


def test_choices_that_dealing_changes_gain():
    """profiles/spmm_plan_equal_parts_slabs.csv: 0.932 of the time, ten of 113 more than 3 % longer."""
    table = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles", "spmm_plan_equal_parts_slabs.csv")
    rows = list(csv.DictReader(line for line in open(table) if not line.startswith("#")))
    ratio = np.array([float(r["us_equal"]) / float(r["us_slices"]) for r in rows])
    assert len(ratio) >= 100 and np.exp(np.log(ratio).mean()) <= 0.94
    assert (ratio > 1.03).sum() <= 10 and np.sort(ratio)[-2] <= 1.07 and ratio.max() <= 1.15


# (8 CUs, one to an XCD: any grid that its slices do not divide)
@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("N,K,M,tm,variant", [
    (400, 300, 50, 16, 106),        # 7 x 4: few tokens, more weight
    (100, 600, 200, 16, 105),       # 4 x 13: many tokens
    (330, 520, 90, 32, 101),        # 3 x 3
    (390, 600, 70, 64, 104),        # 4 x 2, divided: not dealt
    (520, 1030, 75, 32, 104),       # 5 x 3, ring
    (900, 70, 45, 16, 101),         # 8 x 3, divided: not dealt
])
def test_on_the_cpu(N, K, M, tm, variant):
    build_emu.build()
    res = run_case(N, K, M, 0.8, "s8", "none", tm, variant, cus=8)
    assert res["match"] and res["padding_untouched"], res


@pytest.mark.gpu
@pytest.mark.parametrize("out_type,postop", [("s32", "none"), ("u8", "gelu")])
@pytest.mark.parametrize("N,K,M,tuning,workgroups", PROBLEMS + [(4096, 256, 50, (16, 105), None), (300, 256, 2000, (16, 106), None)])
def test_equal_parts_match_the_oracle(N, K, M, tuning, workgroups, out_type, postop):
    from test_gpu_parity import check_case
    check_case(wl.Case("parts", N, K, M, 0.8, wl.N4K1, out_type, postop, keys=(150, N, K, M)), tuning=tuning)
