"""The float64 form of the fixed-point terms (magic_term) has fewer fraction
bits than the form from 32-bit conversions that it replaced (fixed_term), since
a term must stay below 2^51 units, but rounds the product once where the other
rounded it to float32 first.  Over the ranges of fusion's and the adjoint's
sums its error against exact sums is no larger: at most half a unit a term, and
below the other's in the root mean square."""
import ctypes as C
import math
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def libs(tmp_path_factory):
    out = []
    for name in ("fixed_point", "magic_term"):
        so = str(tmp_path_factory.mktemp("fx") / f"lib{name}.so")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-o", so,
                               os.path.join(HERE, "native", f"{name}_harness.cpp")])
        out.append(C.CDLL(so))
    old, new = out
    old.fixed_term_host.restype = C.c_uint64
    old.fixed_term_host.argtypes = [C.c_float, C.c_float, C.c_float]
    new.magic_term_host.restype = C.c_uint64
    new.magic_term_host.argtypes = [C.c_double, C.c_double, C.c_int]
    return old, new


def _sum(units, f):
    units %= 1 << 64
    return (units - (1 << 64) if units >= 1 << 63 else units) / 2.0 ** f


def _errors(libs, pairs, f_old, f_new, product=False):
    """Errors of the sum of w x in both forms.  `product`: the replaced form
    took the float32 product as its term."""
    old, new = libs
    a = b = 0
    for w, x in pairs:
        wo, xo = (np.float32(1.0), w * x) if product else (w, x)
        ws = float(wo) * 2.0 ** f_old
        a += old.fixed_term_host(ws, ws * 2.0 ** -32, float(xo))
        b += new.magic_term_host(float(w), float(x), f_new)
    exact = math.fsum(float(w) * float(x) for w, x in pairs)
    e_new = abs(_sum(b, f_new) - exact)
    assert e_new <= len(pairs) * 2.0 ** -(f_new + 1) + 2.0 ** -52 * abs(exact)
    return abs(_sum(a, f_old) - exact), e_new


def _rms(e):
    return math.sqrt(sum(x * x for x in e) / len(e))


@pytest.mark.parametrize("fx,vs", [(131.0, 0.02), (525.0, 0.01), (525.0, 0.005), (1050.0, 0.005)])
def test_fusion_sums(libs, fx, vs):
    rng = np.random.default_rng(int(fx / vs))
    T = 5 * vs
    side = fx * vs * math.sqrt(3.0) / max(0.4 - T, vs) + 2.0   # of a voxel's footprint, pixels
    f_old = min(56, math.floor(62 - math.log2(side * side)))
    f_new = math.floor(min(62 - math.log2(side * side), 50))
    errors = {"d": [], "n": []}
    for _ in range(100):
        n = int(2 ** rng.uniform(0, 7))
        d = np.clip(rng.uniform(-T, T) + rng.normal(0, 0.003, n), -T, T).astype(np.float32)
        w = np.clip((np.float32(T) - d) * np.float32(1 / (T - vs)), 0, 1).astype(np.float32)
        normal = (0.3 * rng.normal(size=n)).clip(-1, 1).astype(np.float32)
        for k, x in (("d", d), ("n", normal)):
            errors[k].append(_errors(libs, list(zip(w, x)), f_old, f_new))
    for k, e in errors.items():
        old, new = _rms([x for x, _ in e]), _rms([x for _, x in e])
        print(f"{k}: {f_old} bits {old:.1e}, {f_new} bits {new:.1e}")
        assert 0 < new <= old


@pytest.mark.parametrize("n", [1, 8, 100, 3000])
@pytest.mark.parametrize("sigma", [3e-3, 1e-4, 1e-6])
def test_adjoint_sums(libs, n, sigma):
    """n pixels in the block, residuals of sigma metres, Huber threshold 1 cm."""
    rng = np.random.default_rng(n)
    vs, delta = 0.01, 0.01
    ilogb = lambda x: math.frexp(x)[1] - 1
    bound_p = delta
    bound_q = bound_p * (0.5 * vs + 1e-6 * (1.0 + vs * 1e3))
    e = {"psi": [], "g": []}
    for _ in range(60):
        m = max(1, min(n, int(2 ** rng.uniform(0, 5))))
        r = rng.normal(0, sigma, m).clip(-delta, delta).astype(np.float32)
        dq = rng.uniform(-vs / 2, vs / 2, m).astype(np.float32)
        for k, bound, x in (("psi", bound_p, np.ones(m, np.float32)), ("g", bound_q, dq)):
            f_old = min(62, max(0, 61 - ilogb(n * bound)))
            f_new = min(50 - ilogb(bound), 61 - ilogb(n * bound))
            e[k].append(_errors(libs, list(zip(r, x)), f_old, f_new, product=True))
    for k, v in e.items():
        old, new = _rms([x for x, _ in v]), _rms([x for _, x in v])
        print(f"{k}: {old:.1e}, {new:.1e}")
        assert new <= old
