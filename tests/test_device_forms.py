"""The two forms that a weight is uploaded in: written by several threads, read back on the host under the sanitizers, and
exported from the device handle as from a host-only one."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2306_16601_amd as sp

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CXX = shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CXX), reason="no clang++ for a sanitizer build")
@pytest.mark.parametrize("sanitizer", ["address,undefined", "thread"])
def test_forms_hold_the_weight(tmp_path, sanitizer):
    exe, csrc = str(tmp_path / "forms"), os.path.join(ROOT, "paper_2306_16601_amd", "csrc")
    subprocess.run([CXX, "-fsanitize=" + sanitizer, "-fno-sanitize-recover=all", "-g", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "include"),
                    "-I", csrc, os.path.join(csrc, "pack.cpp"), os.path.join(HERE, "sanitize", "device_forms.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout[-500:], r.stderr[-3000:])


@pytest.mark.gpu
@pytest.mark.parametrize("block", ["n4k1", "n1k4"])
@pytest.mark.parametrize("N,K,density", [(1, 1, 1.0), (33, 513, 0.3), (300, 1100, 0.1), (250, 2600, 0.0), (1024, 4096, 0.2)])
def test_a_weight_on_the_device_exports_the_host_only_layout(N, K, density, block):
    rng = np.random.default_rng(N + K)
    W = np.where(rng.random((N, K)) < density, rng.integers(-128, 128, (N, K)), 0).astype(np.int8)
    on_device, host_only = sp.spmm_pack(W, block), sp.spmm_pack_host(W, block)
    try:
        assert sp.spmm_layout_dims(on_device) == sp.spmm_layout_dims(host_only)
        for got, ref in zip(sp.spmm_layout_export(on_device), sp.spmm_layout_export(host_only)):
            assert np.array_equal(np.asarray(got), np.asarray(ref))
        assert np.array_equal(sp.spmm_unpack(on_device), W)
    finally:
        sp.spmm_destroy(on_device)
        sp.spmm_destroy(host_only)
