"""What launches are planned by, the estimates of the resident kernels as they are, against measured times of problems that they
were not fitted to (profiles/spmm_plan_resident_measurements.csv)."""
import csv
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2306_16601_amd as sp

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
TABLE = os.path.join(ROOT, "profiles", "spmm_plan_resident_measurements.csv")
CXX = shutil.which("g++") or shutil.which("clang++")
pytestmark = pytest.mark.skipif(CXX is None, reason="no C++ compiler")

SOURCE = r"""
#include <cstdio>
#include "spmm_internal.h"

int main()
{
    long M, steps, wide_steps;
    int tiles, segments, K, max_segment, max_tile, wide_max, bytes, gelu_f32, sum, aligned;
    while (std::scanf("%ld %d %d %d %ld %d %d %ld %d %d %d %d %d", &M, &tiles, &segments, &K, &steps, &max_segment, &max_tile, &wide_steps,
                      &wide_max, &bytes, &gelu_f32, &sum, &aligned) == 13) {
        const spmm::WeightDims w{tiles, segments, K, steps, max_segment, max_tile, wide_max, wide_steps};
        const spmm::Plan p = spmm::make_plan(M, w, 256, 0, 0, bytes ? 1 : 4, true, true, spmm::wide_tile(gelu_f32, sum),
                                             spmm::wide_handicap(bytes, gelu_f32, sum, aligned));
        if (!p.simple) std::printf("%s%d_%d\n", p.wide ? "WIDE_" : p.loaders ? "FED_" : "", p.token_tile, p.waves);
        else if (p.stream || (p.slab && p.token_tile == 32)) std::printf("RING_%d\n", p.token_tile);
        else if (p.token_tile == 16) std::printf("%s_16w%d\n", p.slab ? "SLAB" : "RES", p.waves);
        else std::printf("RES_%d\n", p.token_tile);
    }
}
"""


@pytest.fixture(scope="module")
def measured(tmp_path_factory):
    """(row of the table, its times, the configuration chosen) of every problem"""
    d = tmp_path_factory.mktemp("plan")
    sp.lib()
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run([CXX, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2306_16601_amd", "csrc"),
                    str(d / "plan.cpp"), sp.binding.LIB_PATH, "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + os.path.dirname(sp.binding.LIB_PATH),
                    "-o", str(d / "plan")], check=True)
    rows = list(csv.DictReader(line for line in open(TABLE) if not line.startswith("#")))
    ask = "".join(" ".join(r[c] for c in ("M", "tiles", "segments", "K", "steps", "max_segment", "max_tile", "wide_steps", "wide_max")) +
                  " %d %d %s %d\n" % (r["out"] in ("s8", "u8"), r["out"] == "f32" and r["post"] == "gelu", r["sum"],
                                      r["layout"] != "packed" or int(r["M"]) % 16 == 0) for r in rows)
    names = subprocess.run([str(d / "plan")], input=ask, capture_output=True, text=True, check=True).stdout.split()
    assert len(names) == len(rows) >= 800
    configurations = list(rows[0])[list(rows[0]).index("before") + 1:]
    out = [(r, {c: float(r[c]) for c in configurations if r[c]}, n) for r, n in zip(rows, names)]
    assert all(n in t and r["before"] in t for r, t, n in out)
    return out


def test_the_times_are_of_the_kernels_that_they_are_listed_for():
    """A weight without the wide form has no times of it: asked for it, it runs 8 compute and 4 loader waves with 128-token tiles."""
    without = 0
    for r in csv.DictReader(line for line in open(TABLE) if not line.startswith("#")):
        wide = [float(r[c]) for c in r if c.startswith("WIDE_") and r[c]]
        without += not wide
        assert bool(wide) == (int(r["wide_max"]) > 0)
        assert len(wide) < 5 or max(wide) > 1.03 * min(wide), r
    assert without >= 20


def test_the_choice_is_close_to_the_fastest_configuration(measured):
    ratio = np.array([t[n] / min(t.values()) for _, t, n in measured])
    assert np.exp(np.log(ratio).mean()) <= 1.015 and (ratio > 1.1).mean() <= 0.035


@pytest.mark.parametrize("layout", ["row", "packed", "tile"])
def test_it_is_better_than_before_in_every_layout(measured, layout):
    gain = np.array([t[r["before"]] / t[n] for r, t, n in measured if r["layout"] == layout])
    assert len(gain) > 150 and np.exp(np.log(gain).mean()) >= 1.01 and (gain < 0.97).mean() <= 0.03
