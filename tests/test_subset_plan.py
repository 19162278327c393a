"""The list builder's rules (csrc/subset_plan.h), compiled for the CPU."""
import os
import subprocess

import numpy as np
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
    assert [r[0] for r in plan([(80768, 1, 1), (80769, 1, 1), (155392, 1, 1), (155393, 1, 1), (201920, 1, 1)])] == [16, 8, 8, 16, 8]


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


def test_slices_without_a_workspace(plan):
    """Half of the workgroups until each of all of them has 65536 tokens; never more than count the stream with a workspace, never none."""
    calls = [(151680, t, 1) for t in (0, 1, 1 << 15, 1 << 18, 1 << 20, (1 << 24) - 1, 1 << 24, (1 << 31) - 1)] + [(250000, (1 << 23) - 1, 1)]
    assert [r[14] for r in plan(calls)] == [8, 8, 8, 64, 128, 128, 256, 256, 64]
    assert all(1 <= r[14] <= r[3] for r in plan([(V, 1 << 20, 1) for V in VOCABS]))


@pytest.fixture(scope="module")
def fields(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fields") / "subset_fields")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wno-unknown-pragmas", "-Werror",
                    os.path.join(ROOT, "tests", "plan", "subset_fields_driver.cpp"), "-o", exe], check=True)
    return lambda bits, V, chunk, toks: subprocess.run([exe, str(bits), str(V), str(chunk)], input=toks.astype(np.int32).tobytes(),
                                                       capture_output=True, check=True).stdout.decode()


@pytest.mark.parametrize("bits", [6, 8, 16])
@pytest.mark.parametrize("V,chunk", [(1000, 1000), (1003, 1003), (1003, 340)])
@pytest.mark.parametrize("kind", ["padded", "out of range", "neighbour", "hot", "all"])
def test_fields_that_wrap_are_counted_exactly(fields, bits, V, chunk, kind):
    """Several widths (also one that leaves bits of a word over), one chunk and several, a last word with fields that have no id; tokens that are not ids of the chunk (padding
    of -1, numbers on both sides of the vocabulary, the id below a chunk's first) wrap nothing that is counted."""
    rng = np.random.default_rng(bits + V + chunk)
    n = 1 << (21 if bits == 16 else 18)
    t = rng.integers(0, V, n)
    if kind == "padded":
        t.reshape(-1, 256)[:, 128:] = -1
    elif kind == "out of range":  # a field of the word that nobody reads and the one above it
        t[rng.random(n) < 0.5] = -1
        t[rng.random(n) < 0.4] = rng.choice([-5, -4, -3, -2, V, V + 1, V + 2, -(1 << 31), (1 << 31) - 1])
    elif kind == "neighbour":
        t[rng.random(n) < 0.9] = min(chunk, V) - 1
    elif kind == "hot":           # whole words full at a time: carries run through several fields
        t[:] = rng.choice([0, 1, 2, 3, 4, 5, 6, 7, V - 3, V - 2, V - 1], n)
    assert fields(bits, V, chunk, t) == ""
