"""Host logic: launch plans with the costs and the largest cut that the library plans its FP64 / FP32,
BF16 and FP8 launches with, pieces starting at any unit (csrc/plan.h), and the rule for the patch rows
of an FP32 launch (csrc/staging.h)."""
import json
import os
import subprocess

import numpy as np
import pytest

from test_launch_plan import CSRC, DRIVER, _case_text, _check_plan

# The driver of the plan tests with the costs named in each case, which are added to the units' work
# and printed.
CALL = "aroam::plan_launch(tu, cs, w, patches, slots, allow != 0, slot_bytes, max_bytes);"
COSTS = r"""
  auto costs = [](int kind) {
    return kind == 0 ? aroam::kRingCosts : kind == 1 ? aroam::kBf16Costs : aroam::kFp8Costs;
  };
  if (argc > 1) {
    for (int kind = 0; kind < 3; ++kind) {
      const aroam::LaunchCosts c = costs(kind);
      std::printf("[%.17g, %.17g, %.17g, %.17g]\n", c.unit, c.plan.workgroup, c.plan.add,
                  c.plan.add_slot);
    }
    std::printf("[%d]\n", aroam::kMaxCut);
    return 0;
  }
  std::string mode;
"""
KINDS = {"ring": 0, "bf16": 1, "fp8": 2}


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    assert CALL in DRIVER and DRIVER.count("  std::string mode;\n") == 1
    d = tmp_path_factory.mktemp("plan_costs")
    src = DRIVER.replace("int main() {", "int main(int argc, char**) {")
    src = src.replace("  std::string mode;\n", COSTS.lstrip("\n"))
    src = src.replace("    const aroam::LaunchPlan p =", "    int kind;\n    std::cin >> kind;\n"
                      "    for (double& x : w) x += costs(kind).unit;\n"
                      "    const aroam::LaunchPlan p =")
    src = src.replace(CALL, CALL.replace("max_bytes);", "max_bytes,\n"
                                         "                           aroam::kMaxCut, costs(kind).plan);"))
    (d / "driver.cpp").write_text(src)
    exe = d / "driver"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC,
                    str(d / "driver.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), "costs"], capture_output=True, text=True, check=True).stdout
    *costs, (max_cut,) = [json.loads(x) for x in out.strip().split("\n")]

    def run(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True,
                             text=True, check=True).stdout
        return [json.loads(x) for x in out.strip().split("\n")]
    return run, costs, max_cut


def layout(rng, n_tiles, most):
    """Tiles of up to `most` units, some empty; a piece may start at every unit."""
    sizes = rng.integers(0, most + 1, size=n_tiles)
    sizes[rng.random(n_tiles) < 0.1] = 0
    units = [0] + list(np.cumsum(sizes).astype(int))
    work = list(rng.integers(1, 60, size=units[-1]) * rng.choice([1.0, 4.0]))
    return units, [list(range(a, b)) for a, b in zip(units, units[1:])], work


def steps(max_cut):
    d, out = 1, []
    while d <= max_cut:
        out.append(d)
        d += max(1, d // 4)
    return out


@pytest.mark.parametrize("kind", KINDS)
def test_shipped_plans_satisfy_the_invariants(built, kind):
    run, costs, max_cut = built
    unit, workgroup, add, add_slot = costs[KINDS[kind]]
    assert min(unit, workgroup, add, add_slot) > 0 and max_cut == 64
    rng = np.random.default_rng(KINDS[kind])
    cases, meta = [], []
    for i in range(150):
        tu, cs, work = layout(rng, int(rng.integers(1, 34)), int(rng.choice([6, 60, 400])))
        patches = int(rng.choice([1, 2, 10, 36, 175]))
        slots = int(rng.choice([512, 768]))
        slot_bytes = 8192.0 if kind == "ring" else 32768.0
        limit = float(rng.choice([1 << 30, 32 << 20, 2 << 20, 0]))
        cases.append(_case_text(tu, cs, work, patches, slots, True, slot_bytes, limit)
                     + f" {KINDS[kind]}")
        meta.append((tu, cs, [w + unit for w in work], patches, slots, slot_bytes, limit))
    plans = run(cases)
    sims, deep = [], 0
    for p, (tu, cs, work, patches, slots, slot_bytes, limit) in zip(plans, meta):
        _check_plan(p, tu, cs, work, patches, slot_bytes, limit, True)
        assert p["cut"] in steps(max_cut)
        assert limit > 0 or p["n_slots"] == 0
        deep += p["cut"] > 8
        sims.append(f"sim {len(p['pieces'])} {patches} {slots} "
                    + " ".join(repr(x[4] + workgroup) for x in p["pieces"]))
    assert deep > 10
    for p, sim in zip(plans, run(sims)):
        # the simulated launch with the workgroups' costs, and the launch that adds the slots
        slots = add + add_slot * max(p["tile_pieces"]) if p["n_slots"] else 0.0
        assert p["time"] == pytest.approx(sim["time"] + slots, rel=1e-12)


def test_slot_costs_stop_cuts_that_the_slots_would_cost_more_than(built):
    """One tile of 64 units on 768 places: the pieces get shorter with the cut and their slots more;
    the plan's cut is the best of all by the same sum, up to the early exit beyond 1.05 of the best."""
    run, costs, max_cut = built
    for kind, (unit, workgroup, add, add_slot) in zip(KINDS, costs):
        for w in (1.0, 20.0, 300.0):
            p, = run([_case_text([0, 64], [list(range(64))], [w] * 64, 1, 768, True) +
                      f" {KINDS[kind]}"])
            whole = 64 * (w + unit) + workgroup
            time = {1: whole}
            for d in steps(max_cut)[1:]:
                sizes = [round(64 * (k + 1) / d) - round(64 * k / d) for k in range(d)]
                time[d] = max(sizes) * (w + unit) + workgroup + add + add_slot * d
            best = min(t for t in time.values() if t == whole or t < 0.9 * whole)
            assert best <= p["time"] * (1 + 1e-12)
            # a cut lands on the nearest unit: up to one unit more than an even share
            assert p["time"] <= best + (w + unit)


def test_pieces_never_exceed_the_rows_of_a_grid(built):
    """2000 tiles of 64 units of nearly free slots: 64 pieces each would be 128 000 rows."""
    run, _, _ = built
    n = 2000
    units = list(range(0, 64 * n + 1, 64))
    p, = run([_case_text(units, [list(range(a, a + 64)) for a in units[:-1]], [1e6] * (64 * n), 1,
                         200000, True, 1.0, 1e18) + " 0"])
    assert 8 < p["cut"] and 16384 < len(p["pieces"]) <= 65535


@pytest.fixture(scope="module")
def ring_rows(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "rows.cpp").write_text(
        '#include "staging.h"\n#include <cstdio>\n#include <cstdlib>\n'
        "int main(int, char** v) {\n"
        '  std::printf("%d", aroam::ring_rows(atoi(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]), '
        "atoi(v[5])));\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "rows.cpp"), "-o",
                    str(d / "rows")], check=True)

    def rule(*a):
        return int(subprocess.run([str(d / "rows"), *map(str, a)], capture_output=True, text=True,
                                  check=True).stdout)
    return rule


def test_patch_rows_rule(ring_rows):
    """Eight rows where the LDS holds two rings of eight but not three of four, and the launch has
    four workgroups per CU."""
    row = lambda k: -(-(32 + 2 * k) * 48 // 256) * 256
    for k in range(0, 98):
        lds = 160 * 1024
        wide = 3 * 11 * row(k) > lds and 2 * 15 * row(k) <= lds
        assert wide == (35 <= k <= 40)
        assert ring_rows(k, 11, 320, 80, 256) == (8 if wide else 4)  # 100 patches
        assert ring_rows(k, 10, 320, 80, 256) == 4
