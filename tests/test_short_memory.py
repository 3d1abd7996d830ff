"""Packing when memory is short: the second form of a weight is not needed to run it, so that a pack fails only where the first
one does not fit, and gives everything back then."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, os.path.join(HERE, "emu"))
import build_emu  # noqa: E402

CXX = shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"


def pack_and_run(N, K, failing, pending=0, copies=0):
    build_emu.build()
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_short_memory.py"), str(N), str(K), str(failing), str(pending), str(copies)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.strip().splitlines()[-1])


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("N,K,failing", [(64, 600, 0b1), (800, 1100, 0b10)])       # one allocation of both forms; two
def test_a_weight_is_packed_when_only_its_first_form_fits(N, K, failing):
    whole, res = pack_and_run(N, K, 0), pack_and_run(N, K, failing)
    assert whole["match"] and "smfmac" in whole["kernel"] and whole["device_bytes"] == whole["both"] and whole["left"] == 0
    assert "error" not in res, res
    assert res["match"] and res["unpacked"] and res["left"] == 0
    assert "smfmac" not in res["kernel"] and 0 < res["device_bytes"] < res["both"]


@pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")
@pytest.mark.parametrize("N,K,failing", [(64, 600, 0b11), (800, 1100, 0b1)])
def test_a_pack_without_memory_for_the_first_form_fails_and_gives_all_back(N, K, failing):
    res = pack_and_run(N, K, failing)
    assert "allocation failed" in res["error"] and res["left"] == 0


@pytest.mark.skipif(not os.path.exists(CXX), reason="no clang++ for a sanitizer build")
def test_the_first_form_is_whole_when_the_host_has_no_memory_for_the_second(tmp_path):
    exe, csrc = str(tmp_path / "memory"), os.path.join(ROOT, "paper_2306_16601_amd", "csrc")
    subprocess.run([CXX, "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-g", "-O1", "-std=c++17", "-pthread", "-I",
                    os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "pack.cpp"),
                    os.path.join(HERE, "sanitize", "short_memory.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout[-500:], r.stderr[-3000:])
