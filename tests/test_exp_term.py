"""The terms of the cross-entropy's sums and the attention's weights (csrc/exp_term.h), compiled for the CPU, against 64 bits."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_weight_of_the_attention_is_right_whatever_its_exponent(tmp_path):
    """A single weight can carry an output (the maximum's split has no token but one, a merge puts two splits together): within two
    units of 2^-24; the terms of long sums are off by up to 2^-24 |t|, 4e-6 here."""
    exe = str(tmp_path / "exp")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wall", "-Werror",
                    os.path.join(ROOT, "tests", "plan", "exp_driver.cpp"), "-o", exe], check=True)
    worst, one, none = map(float, subprocess.run([exe, "weight"], capture_output=True, text=True, check=True).stdout.split())
    assert worst <= 2.0 * 2.0 ** -24 and (one, none) == (1.0, 0.0)


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
