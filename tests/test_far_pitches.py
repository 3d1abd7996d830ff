"""Rows 2^40 elements apart, the largest pitch the library takes, run on the CPU (see tests/test_emulated_kernels.py)."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "emu"))
import build_emu  # noqa: E402

pytestmark = pytest.mark.skipif(not build_emu.available(), reason="no host clang++ for the emulation build")


@pytest.mark.parametrize("out_type, with_sum", [("s8", 0), ("f32", 1)])
def test_rows_two_to_the_forty_elements_apart(out_type, with_sum):
    build_emu.build()
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "run_far_pitch.py"), out_type, str(with_sum)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert json.loads(r.stdout.strip().splitlines()[-1])["match"]
