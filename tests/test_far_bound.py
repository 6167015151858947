"""The far filter's cut-off term bounds what the three harmonics leave out (CPU).

With e(psi) the remainder of (|a + s| - |a|) / |s| = ((1 + 2 x cos psi + x^2)^1/2 - 1) / x
after the harmonics, and its best constant taken out, every weight is within a
factor exp(+-ln 2 |e| |nb s|), so a value of the normalised CDF moves by at most
ln 2 / 2 max |e| |nb s|.  kFarCut x^3 must not be smaller, for every x that the
filter takes.
"""
import os
import re

import numpy as np

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2603_01122_amd", "csrc", "common.hpp")


def constant(name):
    return float(re.search(rf"constexpr float {name} = ([0-9.]+)f;", open(SRC).read()).group(1))


def test_cut_off_term_is_a_bound():
    x_max, cut = constant("kFarX"), constant("kFarCut")
    psi = np.linspace(0.0, 2.0 * np.pi, 8193)
    for x in np.linspace(0.01, x_max, 45):
        f = (np.sqrt(1.0 + 2.0 * x * np.cos(psi) + x * x) - 1.0) / x
        g = ((1.0 - x * x / 8.0) * np.cos(psi) - x / 4.0 * np.cos(2.0 * psi)
             + x * x / 8.0 * np.cos(3.0 * psi))
        e = f - g
        assert 0.5 * np.log(2.0) * 0.5 * (e.max() - e.min()) <= cut * x ** 3, x
