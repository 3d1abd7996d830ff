"""When the plan takes the wide form, against measured launch times (profiles/spmm_plan_wide_measurements.csv): it is asked for
every problem of the table with and without that form, and what it picks is compared with the fastest of what was measured."""
import csv
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2306_16601_amd as sp

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
TABLE = os.path.join(ROOT, "profiles", "spmm_plan_wide_measurements.csv")
CXX = shutil.which("g++") or shutil.which("clang++")
pytestmark = pytest.mark.skipif(CXX is None, reason="no C++ compiler")

SOURCE = r"""
#include <chrono>
#include <cstdio>
#include <vector>
#include "spmm_internal.h"

static void name(const spmm::Plan& p)
{
    if (p.wide) std::printf("WIDE_%d_%d\n", p.token_tile, p.waves);
    else if (!p.simple) std::printf("%s%d_%d\n", p.loaders ? "FED_" : "", p.token_tile, p.waves);
    else if (p.stream || (p.slab && p.token_tile == 32)) std::printf("RING_%d\n", p.token_tile);
    else if (p.token_tile == 16) std::printf("%s_16w%d\n", p.slab ? "SLAB" : "RES", p.waves);
    else std::printf("RES_%d\n", p.token_tile);
}

int main()
{
    long M, steps, wide_steps;
    int tiles, segments, K, max_segment, max_tile, wide_max, bytes, gelu_f32, sum, aligned;
    struct Ask { long M; spmm::WeightDims w; int out_bytes, widest; double handicap; };
    std::vector<Ask> asked;
    while (std::scanf("%ld %d %d %d %ld %d %d %ld %d %d %d %d %d", &M, &tiles, &segments, &K, &steps, &max_segment, &max_tile, &wide_steps, &wide_max,
                      &bytes, &gelu_f32, &sum, &aligned) == 13) {
        const spmm::WeightDims w{tiles, segments, K, steps, max_segment, max_tile, wide_max, wide_steps};
        asked.push_back({M, w, bytes ? 1 : 4, spmm::wide_tile(gelu_f32, sum), spmm::wide_handicap(bytes, gelu_f32, sum, aligned)});
    }
    auto without = [](spmm::WeightDims w) { w.wide_max_steps = 0; w.wide_nsteps = 0; return w; };
    auto plan = [](const Ask& a, const spmm::WeightDims& w) { return spmm::make_plan(a.M, w, 256, 0, 0, a.out_bytes, true, true, a.widest, a.handicap); };
    for (const Ask& a : asked) {
        name(plan(a, a.w));
        name(plan(a, without(a.w)));
    }
    // time of all plans, with and without the form
    double best[2] = {1e9, 1e9};
    long workgroups = 0;
    for (int round = 0; round < 60; ++round)
        for (int with = 0; with < 2; ++with) {
            const auto t = std::chrono::steady_clock::now();
            for (const Ask& a : asked) workgroups += plan(a, with ? a.w : without(a.w)).workgroups;
            const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count() * 1e6;
            if (us < best[with]) best[with] = us;
        }
    std::printf("%f %f %ld\n", best[0] / asked.size(), best[1] / asked.size(), workgroups);
}
"""


def few_blocks(r):
    """The plan does not weigh the wide form (the last rows of the table)."""
    return (int(r["N"]) + 31) // 32 * ((int(r["M"]) + 31) // 32) < 192


@pytest.fixture(scope="module")
def all_asked(tmp_path_factory):
    return choices(TABLE, tmp_path_factory.mktemp("plan"))


@pytest.fixture(scope="module")
def asked(all_asked):
    rows, without, with_it = all_asked
    return [(r, c) for r, c in rows if not few_blocks(r)], without, with_it


def choices(table, d):
    """([row, choice], us of a plan without the wide form, with it)"""
    sp.lib()
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run([CXX, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2306_16601_amd", "csrc"),
                    str(d / "plan.cpp"), sp.binding.LIB_PATH, "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + os.path.dirname(sp.binding.LIB_PATH),
                    "-o", str(d / "plan")], check=True)
    rows = list(csv.DictReader(line for line in open(table) if not line.startswith("#")))
    ask = "".join("%s %s %s %s %s %s %s %s %s %d %d %s %d\n" % (
        r["M"], r["tiles"], r["segments"], r["K"], r["steps"], r["max_segment"], r["max_tile"], r["wide_steps"], r["wide_max"], r["out"] in ("s8", "u8"),
        r["out"] == "f32" and r["post"] == "gelu", r["sum"], r["layout"] != "packed" or int(r["M"]) % 16 == 0) for r in rows)
    lines = subprocess.run([str(d / "plan")], input=ask, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(lines) == 2 * len(rows) + 1
    without, with_it, _ = (float(v) for v in lines[-1].split())
    assert not any(lines[2 * i].startswith("WIDE") for i, r in enumerate(rows) if few_blocks(r) or int(r["wide_max"]) == 0)
    for i, r in enumerate(rows):        # what the plan takes without the form, and its time
        r["other"], r["OTHER"] = lines[2 * i + 1], r[lines[2 * i + 1]]
    return [(r, lines[2 * i]) for i, r in enumerate(rows) if int(r["wide_max"])], without, with_it


def times(r):
    return {k: float(v) for k, v in r.items() if v and (k == "OTHER" or k.startswith("WIDE_"))}


def mean(ratios):
    return float(np.exp(np.log(ratios).mean()))


def test_the_table_has_the_problems(asked):
    assert len(asked[0]) >= 690


def test_short_launches_lose_nothing_without_it(all_asked):
    """With fewer blocks than the plan weighs the form for, no launch that the host does not bound (3.5 us each, and up to 1 us of
    latencies beside it) would be more than 3 % faster."""
    t = [times(r) for r, _ in all_asked[0] if few_blocks(r)]
    assert len(t) >= 150 and all(min(x.values()) >= x["OTHER"] / 1.03 for x in t if x["OTHER"] > 4.8)


def test_the_wide_form_is_taken_where_it_is_faster(asked):
    """Measured on the table: 1.059 times as fast as without the form (1.064 if every choice were right), 0.4 % of the problems
    more than 3 % slower; the choice 1.005 of the fastest one's time, 1.6 % of them over 1.1."""
    gain, off = [], []
    for r, choice in asked[0]:
        t = times(r)
        mine = t[choice if choice.startswith("WIDE") else "OTHER"]
        gain.append(t["OTHER"] / mine)
        off.append(mine / min(t.values()))
    gain, off = np.array(gain), np.array(off)
    assert mean(gain) >= 1.055 and (gain < 1 / 1.03).mean() <= 0.006, (mean(gain), (gain < 1 / 1.03).mean())
    assert mean(off) <= 1.006 and (off > 1.1).mean() <= 0.020, (mean(off), (off > 1.1).mean())


@pytest.mark.parametrize("field, values", [("out", ("s32", "f32", "s8", "u8")), ("layout", ("row", "packed", "tile")), ("block", ("n4k1", "n1k4"))])
def test_it_gains_in_every_type_layout_and_orientation(asked, field, values):
    for v in values:
        gain = [times(r)["OTHER"] / times(r)[c if c.startswith("WIDE") else "OTHER"] for r, c in asked[0] if r[field] == v]
        assert len(gain) >= 30 and mean(gain) >= 1.04, (v, len(gain), mean(gain))


def test_weighing_it_costs_little_of_a_launch(asked):
    """(A plan is made on every launch of 4 us and more.  0.21 us with the form, 0.11 without.)"""
    _, without, with_it = asked
    assert with_it < 3 * without, (with_it, without)
