"""The rules that give a matrix phase its kernel, tiles and reduction parts (csrc/rows_plan.h), compiled for the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256
PART_FLOATS = 16384 * 4 * 256  # the smallest room for partial sums a workspace has


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "rows_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(ROOT, "tests", "plan", "rows_plan_driver.cpp"),
                    "-o", exe], check=True)

    def ask(calls):
        lines = "\n".join("%d %d %d %d %d %d %d" % (c["K"], -(-c["n"] // 16) * 16, c["rows"], c.get("head", 0),
                                                       c.get("pairs", 0), CUS, PART_FLOATS)
                          for c in calls)
        out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split("\n")
        keys = ("serves", "bm", "bn", "parts", "us")
        return [dict(zip(keys, map(float, l.split()))) for l in out if l]

    return ask


@pytest.mark.parametrize("rows", [2, 5, 16, 17, 33, 64])
@pytest.mark.parametrize("K", [288, 544, 1056, 2080, 4128, 8160])
@pytest.mark.parametrize("n", [1024, 4096, 32768])
def test_a_reduction_of_an_odd_number_of_32s_gets_the_tiles_of_its_neighbours(plan, rows, K, n):
    """Model widths are multiples of 32; the tiles for few rows walk a reduction in steps of 64, the last of them half a step.
    Such a call is estimated, and cut, like the next whole number of steps."""
    odd, even = plan([dict(K=K, n=n, rows=rows), dict(K=K + 32, n=n, rows=rows)])
    assert odd["bm"] <= max(16, 2 * rows)
    assert odd["us"] <= even["us"] * 1.001
