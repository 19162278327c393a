"""The rotary factors (csrc/rope.h), compiled for the CPU, against 64 bits."""
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
POSITIONS = [0, 1, 2, 3, 7, 100, 719, 4095, 32767, 65537, 131072, 262143]


@pytest.fixture(scope="module")
def factors(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rope") / "rope")
    # (no fused multiply-adds but the written ones)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wall", "-Werror",
                    os.path.join(ROOT, "tests", "plan", "rope_driver.cpp"), "-o", exe], check=True)

    def ask(pairs):
        text = "\n".join("%d %.17g" % p for p in pairs)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return np.array([[float(x) for x in l.split()] for l in out.split("\n") if l])

    return ask


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("theta", [1e-7, 1e-4, 0.5, 1.0, 1e4, 1e6, 1e9])
def test_rotary_factors(factors, theta, hd):
    """Every theta a handle accepts, positions up to the largest capacity: below a theta of one the angles pass 2^31 quarter
    turns.  Reference: the exact factors of the rounded product.  Bounds: one rounding to float (2^-25 relative to 1), 1e-11 of the
    polynomials, and what the reduction in double leaves (half a unit of the number of quarter turns); the library's functions add
    the rounding of the reduced angle, up to pi, to float."""
    theta = float(np.float32(theta))
    pairs = [(pos, math.pow(theta, -2.0 * j / hd)) for pos in POSITIONS for j in range(hd // 2)]
    got = factors(pairs)
    ang = [pos * inv for pos, inv in pairs]
    want = np.array([[math.cos(a), math.sin(a)] for a in ang])
    turns = np.array(ang) / (math.pi / 2)
    assert (turns.max() > 2 ** 31) == (theta < 1e-5)
    slack = 2.0 ** -25 + 1.1e-11 + 2.0 ** -52 * turns * 1e-3
    assert (np.abs(got[:, :2] - want).max(axis=1) <= slack).all()
    assert (np.abs(got[:, 2:] - want).max(axis=1) <= slack + 2.0 ** -23 + 2.0 ** -24).all()
