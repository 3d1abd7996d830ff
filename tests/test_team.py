"""Threads of a pack (csrc/team.h): passes after the one that was to be the last are shared as those before it."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CXX = shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CXX), reason="no clang++ for a sanitizer build")
@pytest.mark.parametrize("sanitizer", ["address,undefined", "thread"])
def test_threads_are_there_again_after_the_last_pass(tmp_path, sanitizer):
    exe, csrc = str(tmp_path / "team"), os.path.join(ROOT, "paper_2306_16601_amd", "csrc")
    subprocess.run([CXX, "-fsanitize=" + sanitizer, "-fno-sanitize-recover=all", "-g", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "include"),
                    "-I", csrc, os.path.join(csrc, "pack.cpp"), os.path.join(HERE, "sanitize", "team_again.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout[-500:], r.stderr[-3000:])
