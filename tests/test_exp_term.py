"""The terms of the cross-entropy's sums (csrc/exp_term.h), compiled for the CPU, against 64 bits."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("spread", [0.5, 1.3, 3.0])
def test_the_terms_of_a_sum_are_not_off_the_same_way(tmp_path, spread):
    """A term t is off by the rounding of its exponent (2^-24 |t| log2 e) and of exp2 (2^-24), at random: over the 1e4 and more terms
    that carry the sum that averages out to below 1e-8; a constant that is rounded once shifts them all by 2.7 to 6.1e-8 here."""
    exe = str(tmp_path / "exp")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wall", "-Werror",
                    os.path.join(ROOT, "tests", "plan", "exp_driver.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], input="\n".join(f"{seed} {spread}" for seed in range(8)), capture_output=True, text=True,
                         check=True).stdout.split()
    assert [float(v) for v in out[8:]] == [1.0, 0.0]
    assert abs(np.mean([float(v) for v in out[:8]])) < 1e-8, out
