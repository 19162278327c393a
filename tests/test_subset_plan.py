"""The list builder's rules (csrc/subset_plan.h), compiled for the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("subset") / "subset_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(ROOT, "tests", "plan", "subset_plan_driver.cpp"),
                    "-o", exe], check=True)

    def ask(calls):
        lines = "\n".join("%d %d %d" % c for c in calls)
        out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split("\n")
        return [list(map(int, l.split())) for l in out if l]

    return ask


VOCABS = [1, 2, 7, 4096, 80768, 80769, 151680, 155392, 155393, 200001, 201920, 201921, 262144, 403840, 403841, 1000003,
          (1 << 31) - 1 - 4096]


def test_chunks_cover_the_vocabulary_and_fit_a_compute_unit(plan):
    for V, r in zip(VOCABS, plan([(V, 1 << 20, 1) for V in VOCABS])):
        bits, chunks, ids, slices, lds, stream = r[:6]
        assert chunks * ids >= V and (chunks - 1) * ids < V, (V, r)       # the last chunk is not empty
        assert ids % (4 * (32 // bits)) == 0 and lds <= 160 * 1024, (V, r)
        assert 1 <= slices and slices * chunks <= max(256, chunks) and 1 <= stream <= slices, (V, r)
    assert [r[0] for r in plan([(80768, 1, 1), (80769, 1, 1), (155392, 1, 1), (155393, 1, 1), (201920, 1, 1)])] == [16, 8, 8, 6, 6]


def test_the_digits_cover_every_count_the_cut_can_fall_on(plan):
    calls = [(151680, t, n) for t in (0, 1, 7, 4094, 4095, 1 << 24, (1 << 24) + 1, (1 << 31) - 1) for n in (0, 1, 3, 32768, 151680)]
    for (V, t, n), r in zip(calls, plan(calls)):
        cap, passes, digits = r[6], r[7], list(zip(r[8::2], r[9::2]))
        if n == 0:
            assert passes == 0
            continue
        assert cap == t // n + 1                                          # n ids cannot all occur more often than that
        used = digits[:passes]
        assert 1 <= passes <= 3 and all(1 <= b <= 12 for b, _ in used)
        assert used[-1][1] == 0 and all(hi[1] == lo[0] + lo[1] for hi, lo in zip(used, used[1:]))
        assert cap < 1 << (used[0][0] + used[0][1])
