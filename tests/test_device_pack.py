"""Large weights' device forms are made on the device: the same bytes as the host's, and what a pack does when memory is short."""
import ctypes
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

import paper_2306_16601_amd as sp

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, HERE)
sys.path.insert(0, os.path.join(HERE, "emu"))
import build_emu  # noqa: E402
from test_short_memory import pack_and_run  # noqa: E402

emulated = pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    """The packer's two sources, as the emulation changes them, and the emulation, without the product kernels."""
    build_emu.build()
    out, csrc = tmp_path_factory.mktemp("device_pack"), os.path.join(build_emu.OUT, "src")
    subprocess.run([build_emu.CXX, "-std=c++17", "-O1", "-g", "-w", "-I", os.path.join(HERE, "emu", "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", csrc, "-x", "c++", os.path.join(HERE, "emu", "device_pack.cpp"), os.path.join(csrc, "spmm_pack.hip"),
                    os.path.join(csrc, "pack.cpp"), os.path.join(HERE, "emu", "emu.cpp"), "-lpthread", "-o", str(out / "driver")], check=True)
    return str(out / "driver")


# percent of the blocks kept; the wide form: made without a step more than the lists ask for, with more, with left-over k and
# exchanges (n1k4 at 20 %), not at all (too many steps)
CASES = [
    (1, 1, 100, "n4k1", 0), (33, 513, 30, "n4k1", 0), (64, 512, 20, "n4k1", 20), (95, 1100, 10, "n4k1", 5), (130, 1537, 30, "n4k1", 0),
    (32, 511, 100, "n4k1", 0), (50, 700, 0, "n4k1", 0), (48, 640, 0, "n4k1", 2), (17, 5000, 25, "n4k1", 0), (31, 600, 45, "n4k1", 0),
    (96, 512, 10, "n1k4", 0), (47, 777, 20, "n1k4", 10), (64, 1024, 25, "n1k4", 0), (33, 515, 40, "n1k4", 0), (70, 514, 2, "n1k4", 2)]


@emulated
@pytest.mark.parametrize("N,K,percent,block,jitter", CASES)
def test_the_device_makes_the_bytes_that_the_host_does(driver, N, K, percent, block, jitter):
    r = subprocess.run([driver, str(N), str(K), str(percent), block, str(jitter)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout[-300:], r.stderr[-1000:])


@pytest.fixture(scope="module")
def bytes_on_the_device(tmp_path_factory):
    """The same comparison beside the product library, whose kernels make the forms on the GPU."""
    cxx, out, product = shutil.which("g++") or build_emu.CXX, str(tmp_path_factory.mktemp("device_pack") / "bytes.so"), sp.binding.LIB_PATH
    sp.lib()
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2306_16601_amd", "csrc"), "-I", "/opt/rocm/include", os.path.join(HERE, "emu", "device_pack.cpp"),
                    product, "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + os.path.dirname(product), "-o", out], check=True)
    return ctypes.CDLL(out).device_pack_bytes


@pytest.mark.gpu
@pytest.mark.parametrize("N,K,percent,block,jitter", CASES + [(1024, 4096, 20, "n4k1", 0), (1033, 1021, 30, "n4k1", 20), (1100, 1000, 0, "n4k1", 0),
                                                              (1024, 1025, 10, "n1k4", 5), (2000, 700, 25, "n1k4", 10), (70000, 16, 30, "n4k1", 0)])
def test_the_gpu_makes_the_bytes_that_the_host_does(bytes_on_the_device, N, K, percent, block, jitter):
    import torch
    torch.cuda.init()
    wide_size, steps = ctypes.c_int64(-1), ctypes.c_int64(-1)
    rc = bytes_on_the_device(ctypes.c_int64(N), ctypes.c_int64(K), percent, block == "n4k1", jitter, ctypes.byref(wide_size), ctypes.byref(steps))
    assert rc == 0 and wide_size.value >= 0 and steps.value >= 0, rc


@emulated
@pytest.mark.parametrize("failing,expected", [(0b1, "both"), (0b10, "both"), (0b1010, "first"), (0b11, "none"), (0b110, "none")])
def test_short_memory_on_the_device(failing, expected):
    """The device allocates its scratch, then both forms; where either does not fit, the host packs, which allocates the first form,
    then the wide one.  Without memory for that one the weight has only the first."""
    res = pack_and_run(1024, 1040, failing)
    assert res["left"] == 0
    if expected == "none":
        assert "allocation failed" in res["error"]
        return
    assert "error" not in res and res["match"] and res["unpacked"]
    assert ("smfmac" in res["kernel"]) == (expected == "both") and (res["device_bytes"] == res["both"]) == (expected == "both")


@emulated
@pytest.mark.parametrize("copies", [0b1, 0b10, 0b100])           # of the weight, of the numbers of steps, of what stands before the records
def test_a_copy_without_memory_leaves_nothing_behind(copies):
    """The host packs then, into an allocation of its own."""
    res = pack_and_run(1024, 1040, 0, copies=copies)
    assert "error" not in res and res["match"] and res["unpacked"] and res["device_bytes"] == res["both"] and res["left"] == 0, res


@emulated
@pytest.mark.parametrize("N,K", [(1024, 1040), (64, 600)])        # forms made by the device, by the host
def test_an_error_left_by_an_earlier_call_is_not_the_pack_s(N, K):
    """600: the runtime's answer to a query of an event that is not over, say.  The pack neither takes it for its own nor takes it away."""
    res = pack_and_run(N, K, 0, pending=600)
    assert "error" not in res and res["match"] and res["unpacked"] and res["device_bytes"] == res["both"] and res["error_left"] == 600, res


@pytest.mark.gpu
@pytest.mark.parametrize("N,K,density,block", [(1024, 1024, 0.2, "n4k1"), (1033, 1021, 0.1, "n4k1"), (257, 4096, 0.3, "n4k1"), (1024, 1025, 0.1, "n1k4"),
                                               (1100, 1000, 0.0, "n4k1")])
def test_a_weight_packed_on_the_device_runs(N, K, density, block):
    """Exact accumulators over both forms, and the weight handed back; rows that do not lie back to back take the host's way."""
    import torch
    rng = np.random.default_rng(N + K)
    keep = rng.random((-(-N // 4), K) if block == "n4k1" else (N, -(-K // 4))) < density
    keep = np.repeat(keep, 4, axis=0)[:N] if block == "n4k1" else np.repeat(keep, 4, axis=1)[:, :K]
    W = np.where(keep, rng.integers(-128, 128, (N, K)), 0).astype(np.int8)
    X = rng.integers(0, 256, (K, 70), dtype=np.uint8)
    strided = np.zeros((N, K + 3), dtype=np.int8)
    strided[:, :K] = W
    x, ref = torch.from_numpy(X).cuda(), W.astype(np.int64) @ X.astype(np.int64)
    for weight in (W, strided[:, :K]):
        h = sp.spmm_pack(weight, block)
        try:
            assert np.array_equal(sp.spmm_unpack(h), W)
            variants = [(0, 0), (16, 101), (32, 101), (64, 104)] + ([(32, 134), (64, 134)] if density else [])
            for tuning in variants:
                sp.spmm_set_tuning(h, *tuning)
                out = torch.full((N, 70), -1, dtype=torch.int32, device="cuda")
                sp.spmm_run(h, x, 70, 70, sp.make_epilogue(None, 1.0, 0, None, "none", "s32"), out, 70, torch.cuda.current_stream().cuda_stream)
                assert np.array_equal(out.cpu().numpy(), ref), tuning
        finally:
            sp.spmm_destroy(h)


@pytest.mark.gpu
def test_a_pack_does_not_wait_for_other_streams():
    """A model's next weight is packed beside work that is under way on streams of its own."""
    import torch
    W = np.where(np.random.default_rng(1).random((1024, 1024)) < 0.2, 3, 0).astype(np.int8)
    a, b = torch.zeros((2, 8192, 8192), dtype=torch.bfloat16, device="cuda")
    other = torch.cuda.Stream()
    with torch.cuda.stream(other):
        torch.mm(a, a, out=b)
    sp.spmm_destroy(sp.spmm_pack(W))
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        for _ in range(200):            # (150 ms; a pack takes 0.2)
            torch.mm(a, a, out=b)
    end = other.record_event()
    h = sp.spmm_pack(W)
    under_way = not end.query()
    torch.cuda.synchronize()
    try:
        assert under_way and np.array_equal(sp.spmm_unpack(h), W)
    finally:
        sp.spmm_destroy(h)


@pytest.mark.gpu
def test_a_pack_keeps_no_scratch():
    """What is gone from the device's free memory when the call returns are the forms (in pages of up to 2 MB, an allocation each)."""
    import torch
    W = np.where(np.random.default_rng(2).random((4096, 4096)) < 0.05, 5, 0).astype(np.int8)
    sp.spmm_destroy(sp.spmm_pack(W))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    h = sp.spmm_pack(W)
    try:
        assert before - torch.cuda.mem_get_info()[0] <= sp.spmm_info(h)[4] + 4 * 2 ** 20
    finally:
        sp.spmm_destroy(h)
