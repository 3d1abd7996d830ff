"""The short-batch kernels that keep all of K in LDS: every number of passes of activation rows and one row more, rows cut by the
end of the matrix in each of them, row-major and tile-major, weights whose tiles are uneven but placed or too uneven for that, Sum, K
in rounds, activations that span gibibytes."""
import os
import sys

import numpy as np
import pytest

import paper_2306_16601_amd as sp
import workloads as wl

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "emu"))
import build_emu  # noqa: E402
from test_emulated_kernels import run_case  # noqa: E402

# (token tile, variant, rows of a pass, resident rows)
KERNELS = [(16, 101, 512, 2048), (16, 105, 512, 2048), (32, 106, 256, 2048), (32, 101, 256, 2048), (64, 101, 128, 1024), (64, 102, 128, 1024),
           (16, 103, 512, 4096), (16, 106, 512, 4096)]


def ks(rows, resident):
    passes = [1, 2, 3, 4, 5, 8]
    return sorted({k for p in passes if p * rows <= resident for k in (p * rows, p * rows + 1)} | {3, resident - 1, resident, resident + 1})


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("tm,variant,K,M,kind", [
    (16, 101, 513, 21, "uniform"), (16, 105, 1025, 37, "ragged"), (32, 106, 257, 45, "uniform"), (32, 101, 1030, 70, "ragged"),
    (64, 101, 129, 67, "uniform"), (64, 102, 1025, 65, "ragged"), (16, 106, 2600, 29, "uniform"), (16, 103, 4097, 17, "ragged")])
def test_on_the_cpu(tm, variant, K, M, kind):
    build_emu.build()
    res = run_case(144, K, M, 0.8, "s8", "none", tm, variant, kind=kind)
    assert res["match"] and res["padding_untouched"], res


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("tm,variant,K,group", [(16, 101, 2048, 4), (32, 101, 2048, 2), (64, 101, 1024, 2), (64, 102, 1024, 2), (16, 103, 4096, 4)])
def test_steps_that_a_tile_does_not_have_are_not_multiplied(tm, variant, K, group):
    """Steps are requested up to the longest tile's number, before the bounds have arrived.  The ring multiplies just those that
    there are; the resident kernels whole groups of them, and no more."""
    build_emu.build()
    N, M = 160, 50
    res, ring = (run_case(N, K, M, 0.7, "s32", "none", tm, v, kind="uneven") for v in (variant, 104))
    assert res["match"] and ring["match"], (res, ring)
    slack = N // 16 * (group - 1) * -(-M // tm) * tm // 16
    assert ring["products"] <= res["products"] <= ring["products"] + slack, (res, ring)


@pytest.mark.gpu
@pytest.mark.parametrize("tm,variant,rows,resident", KERNELS)
def test_passes_on_the_device(tm, variant, rows, resident):
    from test_gpu_parity import check_case
    outs = [("s32", "none"), ("f32", "none"), ("u8", "gelu"), ("s8", "none")]
    for i, K in enumerate(ks(rows, resident)):
        out_type, postop = outs[i % 4]
        M = tm * (1 + i % 2) + (i * 5) % tm + 1
        case = wl.Case("resident", 80 + 16 * (i % 5), K, M, 0.8, wl.N4K1, out_type, postop, keys=(130, K, M))
        check_case(case, tuning=(tm, variant))
        check_case(case, tuning=(tm, variant), ldx=M + 3, ldo=M + 5)


def thinned(d, kind):
    """Row tiles of very different lengths: one 1.3 times as long as the others, or step lists too uneven for a fixed place."""
    W = d["W"] = d["W"].copy()
    if kind == "uneven":
        W[16:, W.shape[1] - W.shape[1] // 4:] = 0
    elif kind == "ragged":
        W[16:64] = 0
        W[64:, :max(0, W.shape[1] - 300)] = 0
    return d


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("tm,variant,K", [(16, 105, 520), (16, 103, 2100), (32, 101, 700), (64, 101, 300), (64, 102, 650)])
def test_tile_major_and_sum_on_the_cpu(tm, variant, K):
    """Rows past K, which the last pass of activations has, lie in the next token tile, or past the end of an exactly sized
    allocation; N is no multiple of 16, and Sum's operand has nothing behind its last value."""
    build_emu.build()
    for args in (dict(xtiled=True, kind="uneven"), dict(xtiled="out"), dict(ld_sum=51)):
        res = run_case(83, K, 45, 0.8, "s8", "none", tm, variant, **args)
        assert res["match"] and res["padding_untouched"], (args, res)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["uniform", "uneven", "ragged"])
@pytest.mark.parametrize("tm,variant,rows,resident", KERNELS)
def test_weights_layouts_and_sum_on_the_device(tm, variant, rows, resident, kind):
    from test_gpu_parity import _run_sum, assert_parity, gpu_spmm, oracle_spmm
    import oracle
    for i, K in enumerate((rows + 1, resident - resident // 4, resident // 2 + 1, resident)):
        N, M = 83, tm * 2 + 5 + i
        for out_type, postop in (("s32", "none"), ("u8", "gelu")):
            case = wl.Case("resident", N, K, M, 0.8, wl.N4K1, out_type, postop, keys=(132, K, M))
            d = thinned(wl.make(case), kind)
            ref = oracle_spmm(d["W"], d["X"], d, case)
            for x_tiled in (False, True):
                got, guards_ok = gpu_spmm(d["W"], d["X"], d, case, tuning=(tm, variant), x_tiled=x_tiled)
                assert guards_ok
                assert_parity(got, ref, case)
        for out_type in ("f32", "s8"):
            case = wl.Case("resident", N, K, M, 0.8, wl.N4K1, out_type, "none", keys=(133, K, M))
            d = thinned(wl.make(case), kind)
            R = (wl.rng_for(134, N, M).standard_normal((N, M)) * wl.preact_sigma(K, case.sparsity)).astype(np.float32)
            ref = oracle.spmm(d["W"], d["X"], d["w_scale"], d["x_scale"], d["bias"], "none", out_type, d["out_scale"],
                              d["out_zero_point"], d["mid_scale"], d["x_zero_point"], sum=R)
            assert_parity(_run_sum(d, case, R, M + i, (tm, variant), i), ref, case)


@pytest.mark.gpu
@pytest.mark.parametrize("tm,variant", [(16, 101), (32, 106), (64, 101)])
def test_activations_beyond_a_gibibyte(tm, variant):
    import torch
    N, K, M, ld = 64, 300, 45, (1 << 22) - 3
    rng = np.random.default_rng(131)
    h = sp.spmm_pack(rng.integers(-127, 128, size=(N, K), dtype=np.int8))
    try:
        x = torch.from_numpy(rng.integers(0, 256, size=(K, M), dtype=np.uint8)).cuda()
        far = torch.empty((K - 1) * ld + M, dtype=torch.uint8, device="cuda")
        far.as_strided((K, M), (ld, 1)).copy_(x)
        ep = sp.make_epilogue(None, 1.0, 0, None, "none", "s32")
        out = [torch.zeros((N, M), dtype=torch.int32, device="cuda") for _ in range(2)]
        sp.spmm_set_tuning(h, tm, variant)
        for X, ldx, o in ((x, M, out[0]), (far, ld, out[1])):
            sp.spmm_run(h, X, M, ldx, ep, o, M, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1]) and out[0].any()
    finally:
        sp.spmm_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("K, M, ld", [
    (601, 262, 3579139),                    # the last 16 bytes at 2^31 - 2, the largest offset of the straight start
    (601, 263, 3579139),                    # ... and at 2^31 - 1, one beyond it
    (1025, 45, (1 << 22) - 3)])             # 4 GiB; one row more than the 64-token kernel keeps
@pytest.mark.parametrize("tm,variant", [(16, 101), (16, 103), (32, 106), (64, 101), (64, 102)])
def test_activations_at_the_last_32_bit_offset(tm, variant, K, M, ld):
    import torch
    N = 83
    rng = np.random.default_rng(131)
    h = sp.spmm_pack(rng.integers(-127, 128, size=(N, K), dtype=np.int8))
    try:
        x = torch.from_numpy(rng.integers(0, 256, size=(K, M), dtype=np.uint8)).cuda()
        far = torch.empty((K - 1) * ld + M, dtype=torch.uint8, device="cuda")
        far.as_strided((K, M), (ld, 1)).copy_(x)
        ep = sp.make_epilogue(None, 1.0, 0, None, "none", "s32")
        out = [torch.zeros((N, M), dtype=torch.int32, device="cuda") for _ in range(2)]
        sp.spmm_set_tuning(h, tm, variant)
        for X, ldx, o in ((x, M, out[0]), (far, ld, out[1])):
            sp.spmm_run(h, X, M, ldx, ep, o, M, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1]) and out[0].any()
    finally:
        sp.spmm_destroy(h)
