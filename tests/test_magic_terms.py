"""The float64 form of the fixed-point terms of fusion's per-frame voxel sums
(gsdf_fixed.hpp, built for the host): w x rounded once to a multiple of 2^-f,
for every magnitude and sign that the kernel's bound |w x| < 2^(51-f) allows."""
import ctypes as C
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def term(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("magic") / "libmagic.so")
    src = os.path.join(HERE, "native", "magic_term_harness.cpp")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-o", out, src])
    lib = C.CDLL(out)
    lib.magic_term_host.restype = C.c_uint64
    lib.magic_term_host.argtypes = [C.c_double, C.c_double, C.c_int]

    def call(w, x, f):
        v = lib.magic_term_host(float(w), float(x), f)
        return v - (1 << 64) if v >= (1 << 63) else v

    return call


@pytest.mark.parametrize("f", [24, 40, 50])
def test_terms_are_the_product_rounded_once(term, f):
    rng = np.random.default_rng(f)
    cases = [(1.0, 1.0), (1.0, -1.0), (0.0, 0.5), (1.0, 0.0), (1.0, 2.0 ** -f), (1.0, -2.0 ** -f), (0.5, 2.0 ** -f),
             (1.0, 2.0 ** (50 - f)), (1.0, -2.0 ** (50 - f))]
    for _ in range(3000):
        w = np.float32(rng.uniform(0.0, 1.0) * 10.0 ** rng.integers(-9, 1))
        x = np.float32(rng.uniform(-1.0, 1.0) * 10.0 ** rng.integers(-9, 1))
        cases.append((float(w), float(x)))
    for w, x in cases:
        exact = Fraction(w) * Fraction(x) * 2 ** f
        assert abs(Fraction(term(w, x, f)) - exact) <= Fraction(1, 2), (w, x, f)
