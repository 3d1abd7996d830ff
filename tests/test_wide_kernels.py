"""The kernels over the wide form (32-row tiles, 2 of every 4 listed k): run on the CPU where tiles, token counts, segments
and step lists have their edges, and on the device in every form against the oracle.  Results are exact: whole numbers
and codes to the bit, f32 to the bit without GELU and within the bound of test_gpu_parity with it."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
import workloads as wl

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "emu"))
import build_emu  # noqa: E402
from test_emulated_kernels import run_case  # noqa: E402

# (N, K, M, sparsity, out, postop, token tile, variant, expected kernel, extra)
EMULATED = [
    # whole tiles; one row over a tile, one k over a segment, one token over a tile; several tiles and segments a stream
    (256, 512, 256, 0.9, "s32", "none", 128, 132, "spmm_rowtile_smfmac<128, 8", {}),
    (257, 513, 129, 0.9, "s8", "gelu", 128, 132, "spmm_rowtile_smfmac<128, 8", {"cus": 2}),
    (320, 1500, 700, 0.8, "s8", "gelu", 96, 132, "spmm_rowtile_smfmac<96, 8", {"cus": 2, "ldx": 704, "ldo": 704}),
    (300, 1100, 333, 0.85, "f32", "none", 96, 132, "spmm_rowtile_smfmac<96, 8", {"cus": 2, "ldo": 336}),
    (260, 1600, 257, 0.9, "f32", "gelu", 64, 132, "spmm_rowtile_smfmac<64, 8", {"cus": 2, "ldx": 261, "ldo": 263}),
    (100, 1100, 203, 0.7, "u8", "none", 64, 134, "spmm_rowtile_smfmac<64, 4", {"cus": 2}),
    (260, 2300, 57, 0.9, "s32", "none", 32, 134, "spmm_rowtile_smfmac<32, 4", {"cus": 2}),
    (33, 3, 7, 0.0, "u8", "gelu", 32, 134, "spmm_rowtile_smfmac<32, 4", {"cus": 2}),
    # rows that use every k: two of a quad is all that fits, so 256 k of a segment have the form and 257 have none
    (40, 256, 40, 0.0, "s32", "none", 32, 134, "spmm_rowtile_smfmac<32, 4", {"cus": 2}),
    (40, 257, 40, 0.0, "s32", "none", 32, 134, "spmm_rowtile_mfma_fed<", {"cus": 2}),
    # more segments than the counts in scalar registers hold
    (72, 8700, 70, 0.9, "s8", "gelu", 64, 134, "spmm_rowtile_smfmac<64, 4", {"cus": 2}),
    # empty segments and tiles, tile-major activations and outputs
    (300, 1700, 200, 0.9, "s32", "none", 96, 132, "spmm_rowtile_smfmac<96, 8", {"cus": 2, "ldo": 208, "kind": "empty"}),
    (300, 1700, 200, 0.9, "s8", "gelu", 32, 134, "spmm_rowtile_smfmac<32, 4", {"cus": 2, "kind": "empty", "xtiled": "out"}),
    (260, 1100, 200, 0.8, "u8", "gelu", 128, 132, "spmm_rowtile_smfmac<128, 8", {"cus": 2, "xtiled": True}),
    # lists of 6 steps
    (289, 1100, 201, 0.86, "s8", "gelu", 128, 132, "spmm_rowtile_smfmac<128, 8, 6", {"cus": 2}),
    (257, 512, 129, 0.85, "f32", "none", 96, 132, "spmm_rowtile_smfmac<96, 8, 6", {"cus": 2, "ldo": 131}),
    (130, 1024, 200, 0.86, "u8", "none", 64, 132, "spmm_rowtile_smfmac<64, 8, 6", {"cus": 2, "xtiled": "out"}),
    (289, 1100, 70, 0.86, "f32", "gelu", 64, 134, "spmm_rowtile_smfmac<64, 4, 6", {"cus": 2}),
    (257, 512, 129, 0.85, "s32", "none", 32, 134, "spmm_rowtile_smfmac<32, 4, 6", {"cus": 2, "ldx": 136}),
    # the operand of Sum, read to its last value and no further
    (257, 513, 129, 0.9, "f32", "none", 64, 132, "spmm_rowtile_smfmac<64, 8", {"cus": 2, "ld_sum": 129}),
    (289, 1100, 70, 0.86, "s8", "none", 64, 134, "spmm_rowtile_smfmac<64, 4, 6", {"cus": 2, "ld_sum": 73, "xtiled": "out"}),
    (100, 1100, 203, 0.7, "u8", "none", 32, 134, "spmm_rowtile_smfmac<32, 4", {"cus": 2, "ld_sum": 208}),
    (64, 600, 128, 0.9, "f32", "none", 128, 132, "spmm_rowtile_smfmac<", {"cus": 2, "ld_sum": 128, "ldo": 128}),
]


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("case", EMULATED, ids=lambda c: "%dx%d_m%d_%s_%s_tm%d_v%d" % (c[0], c[1], c[2], c[4], c[5], c[6], c[7]))
def test_wide_kernel_on_the_cpu_matches_oracle_and_stays_in_bounds(case):
    N, K, M, s, ot, po, tm, var, family, extra = case
    build_emu.build()
    res = run_case(N, K, M, s, ot, po, tm, var, **extra)
    assert family in res["kernel"], res["kernel"]
    assert res["match"], "%d outputs differ from the oracle" % res["mismatches"]
    assert res["padding_untouched"]


TUNINGS = [(128, 132), (96, 132), (64, 132), (64, 134), (32, 134)]
SHAPES = [(31, 100, 33, 0.8), (289, 1100, 701, 0.9), (260, 513, 1299, 0.8), (96, 9000, 130, 0.9), (1024, 1024, 1531, 0.75)]
# 6 step slots in 4x1 blocks, and in 1x4 blocks
SIX = [(289, 1100, 701, 0.86, wl.N4K1), (289, 1100, 701, 0.97, wl.N1K4), (512, 512, 1531, 0.87, wl.N4K1)]
# what the weights of this file's device tests run with: step slots, None = too dense for the form
SLOTS = [(31, 100, 0.8, wl.N4K1, 101, 5), (289, 1100, 0.9, wl.N4K1, 101, 5), (260, 513, 0.8, wl.N4K1, 101, 7), (96, 9000, 0.9, wl.N4K1, 101, 5),
         (1024, 1024, 0.75, wl.N4K1, 101, 8), (31, 100, 0.8, wl.N1K4, 101, 5), (289, 1100, 0.9, wl.N1K4, 101, 8), (260, 513, 0.8, wl.N1K4, 101, 8),
         (96, 9000, 0.9, wl.N1K4, 101, 8), (1024, 1024, 0.75, wl.N1K4, 101, None),
         (31, 100, 0.8, wl.N4K1, 102, 5), (289, 1100, 0.9, wl.N4K1, 102, 5), (260, 513, 0.8, wl.N4K1, 102, 7), (96, 9000, 0.9, wl.N4K1, 102, 5),
         (1024, 1024, 0.75, wl.N4K1, 102, 8)]


KERNELS = """
import json, sys
sys.path[:0] = sys.argv[1:3]
import build_emu, paper_2306_16601_amd.binding as b
b.LIB_PATH = build_emu.LIB
import paper_2306_16601_amd as sp, workloads as wl
for (N, K, M, s, block, key), tunings in json.load(sys.stdin):
    h = sp.spmm_pack(wl.make(wl.Case("slots", N, K, M, s, block, "s8", "gelu", keys=(key, N, K, M)))["W"], block)
    for tuning in tunings:
        sp.spmm_set_tuning(h, *tuning)
        print(sp.spmm_kernel_variant(h, M, "s8", "gelu"))
    sp.spmm_destroy(h)
"""


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
def test_the_device_tests_run_the_kernels_they_name():
    """The step slots of every weight that is run on the device, from the plan over its packed form."""
    build_emu.build()
    tokens = {(N, K, s): M for N, K, M, s in SHAPES}
    cases = [((N, K, tokens[N, K, s], s, block, key), slots) for N, K, s, block, key, slots in SLOTS]
    cases += [((N, K, M, s, block, key), 6) for N, K, M, s, block in SIX for key in (108, 109)]
    here = os.path.dirname(os.path.abspath(__file__))
    r = subprocess.run([sys.executable, "-c", KERNELS, os.path.dirname(here), os.path.join(here, "emu")], text=True, timeout=300, capture_output=True,
                       input=json.dumps([(c, TUNINGS) for c, _ in cases]), env=dict(os.environ, EMU_CUS="256"))
    assert r.returncode == 0, r.stderr[-2000:]
    expected = ["smfmac<%d, %d, %d, 2, 1>" % (tm, 8 if variant == 132 else 4, slots) if slots else "spmm_rowtile_mfma_fed<128, 8, 4, 8, 2, 1>"
                for _, slots in cases for tm, variant in TUNINGS]
    names = r.stdout.splitlines()
    assert len(names) == len(expected)
    for name, want in zip(names, expected):
        assert want in name, (name, want)


@pytest.mark.gpu
@pytest.mark.parametrize("out_type,postop", [("s32", "none"), ("f32", "none"), ("f32", "gelu"), ("s8", "none"), ("u8", "gelu")])
@pytest.mark.parametrize("N,K,M,s,block", SIX)
def test_six_step_slots_on_the_device(N, K, M, s, block, out_type, postop):
    from test_gpu_parity import _run_sum, _run_tiled_out, assert_parity, check_case, oracle_spmm
    case = wl.Case("six", N, K, M, s, block, out_type, postop, keys=(108, N, K, M))
    for i, tuning in enumerate(TUNINGS):
        check_case(case, tuning=tuning, ldx=M + i, ldo=M + 3 * (i % 2))
    if out_type in ("s8", "u8"):
        d = wl.make(case)
        ref = oracle_spmm(d["W"], d["X"], d, case)
        for i, tuning in enumerate(TUNINGS):
            assert_parity(_run_tiled_out(d, case, tuning, i % 2 == 0), ref, case)
    if out_type == "s32" or postop == "gelu":
        return
    case = wl.Case("sixsum", N, K, M, s, block, out_type, postop, keys=(109, N, K, M))
    d = wl.make(case)
    R = (wl.rng_for(110, N, M).standard_normal((N, M)) * wl.preact_sigma(K, case.sparsity)).astype(np.float32)
    ref = oracle.spmm(d["W"], d["X"], d["w_scale"], d["x_scale"], d["bias"], postop, out_type, d["out_scale"], d["out_zero_point"], d["mid_scale"],
                      d["x_zero_point"], sum=R)
    for i, tuning in enumerate(TUNINGS):
        assert_parity(_run_sum(d, case, R, M + i, tuning, i % 4), ref, case)


@pytest.mark.gpu
@pytest.mark.parametrize("out_type,postop", [("s32", "none"), ("f32", "none"), ("f32", "gelu"), ("s8", "none"), ("u8", "gelu")])
@pytest.mark.parametrize("N,K,M,s", SHAPES)
def test_wide_kernels_on_the_device(N, K, M, s, out_type, postop):
    from test_gpu_parity import check_case
    case = wl.Case("wide", N, K, M, s, wl.N4K1, out_type, postop, keys=(101, N, K, M))
    ld = (M + 15) // 16 * 16
    for i, tuning in enumerate(TUNINGS):
        check_case(case, tuning=tuning)
        check_case(case, tuning=tuning, ldx=ld, ldo=ld, x_tiled=i % 2 == 0)
        check_case(case, tuning=tuning, ldx=M + 3, ldo=M + 1 + i, x_offset=3, out_offset=1)
        check_case(case.with_(orientation=wl.N1K4), tuning=tuning)


@pytest.mark.gpu
@pytest.mark.parametrize("out_type", ["s8", "u8"])
@pytest.mark.parametrize("N,K,M,s", SHAPES)
def test_wide_kernels_in_tile_major_order(N, K, M, s, out_type):
    from test_gpu_parity import _run_tiled_out, assert_parity, oracle_spmm
    case = wl.Case("wide", N, K, M, s, wl.N4K1, out_type, "gelu", keys=(101, N, K, M))
    d = wl.make(case)
    ref = oracle_spmm(d["W"], d["X"], d, case)
    for i, tuning in enumerate(TUNINGS):
        assert_parity(_run_tiled_out(d, case, tuning, i % 2 == 0), ref, case)


@pytest.mark.gpu
@pytest.mark.parametrize("out_type,postop", [("f32", "none"), ("s8", "none"), ("u8", "none")])
@pytest.mark.parametrize("N,K,M,s", SHAPES)
def test_wide_kernels_add_their_sum(N, K, M, s, out_type, postop):
    from test_gpu_parity import _run_sum, assert_parity
    case = wl.Case("widesum", N, K, M, s, wl.N4K1, out_type, postop, keys=(102, N, K, M))
    d = wl.make(case)
    R = (wl.rng_for(103, N, M).standard_normal((N, M)) * wl.preact_sigma(K, case.sparsity)).astype(np.float32)
    ref = oracle.spmm(d["W"], d["X"], d["w_scale"], d["x_scale"], d["bias"], postop, out_type, d["out_scale"],
                      d["out_zero_point"], d["mid_scale"], d["x_zero_point"], sum=R)
    for i, tuning in enumerate(TUNINGS):
        assert_parity(_run_sum(d, case, R, M + i, tuning, i % 4), ref, case)


@pytest.mark.gpu
@pytest.mark.parametrize("orient", [wl.N4K1, wl.N1K4])
@pytest.mark.parametrize("density", ["dense rows", "one tile of them", "extremes"])
def test_weights_at_the_limits_of_the_form(orient, density):
    """Rows that use every k have no wide form (three of a quad), and what asks for it runs the form that they have; one
    such block-row among sparse ones; values of -128 and 127 over activations of 255, whose sums are the largest."""
    import paper_2306_16601_amd as sp
    from test_gpu_parity import gpu_spmm, assert_parity
    N, K, M = 96, 1025, 300
    case = wl.Case("limits", N, K, M, 0.9, orient, "s32", "none", keys=(104, N, K, M))
    d = wl.make(case)
    W, X = d["W"].copy(), d["X"]
    if density == "dense rows":
        W[:] = wl.rng_for(105, N, K).integers(-128, 128, size=(N, K), dtype=np.int8)
    elif density == "one tile of them":
        W[32:64] = 1
    else:
        W[W != 0] = np.where(wl.rng_for(106, N, K).integers(0, 2, size=(N, K)) == 1, 127, -128).astype(np.int8)[W != 0]
        X = np.full_like(X, 255)
    ref = oracle.spmm(W, X, d["w_scale"], d["x_scale"], d["bias"], "none", "s32", d["out_scale"], d["out_zero_point"], d["mid_scale"],
                      d["x_zero_point"])
    for tuning in TUNINGS:
        got, guards_ok = gpu_spmm(W, X, d, case, tuning=tuning)
        assert guards_ok
        assert_parity(got, ref, case)
    h = sp.spmm_pack(W, orient)
    try:
        sp.spmm_set_tuning(h, 128, 132)
        assert ("smfmac" in sp.spmm_kernel_variant(h, M, "s32", "none")) == (density == "extremes")
    finally:
        sp.spmm_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("N,K,M,s,out_type", [(2048, 2048, 2048, 0.9, "s8"), (1024, 4096, 1536, 0.8, "s32"), (3000, 2000, 1777, 0.75, "u8")])
def test_the_plans_choice_of_the_wide_form_agrees_with_the_other_kernels(N, K, M, s, out_type):
    """(Sizes with more than two segments, where its estimate is under 0.9 of the others' best.)"""
    import paper_2306_16601_amd as sp
    from test_gpu_parity import gpu_spmm
    case = wl.Case("route", N, K, M, s, wl.N4K1, out_type, "none", keys=(107, N, K, M))
    d = wl.make(case)
    h = sp.spmm_pack(d["W"], case.orientation)
    try:
        assert "smfmac" in sp.spmm_kernel_variant(h, M, out_type, "none")
    finally:
        sp.spmm_destroy(h)
    for pitch in (M, (M + 127) // 128 * 128, M + 5):
        got, ok = gpu_spmm(d["W"], d["X"], d, case, ldx=pitch, ldo=pitch)
        other, ok2 = gpu_spmm(d["W"], d["X"], d, case, ldx=pitch, ldo=pitch, tuning=(128, 108))
        assert ok and ok2 and np.array_equal(got, other)
