"""Effective-action tables and reference actions whose terms leave the FP64 range (host code)."""
import math
import os
import shutil
import subprocess
from fractions import Fraction

import numpy as np
import pytest

import paper_1105_0542_amd as P
from oracle import vector as ov

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1105_0542_amd", "csrc")


@pytest.mark.parametrize("coefs,dim,p", [((0.0, 1e200, 0.0), 1, 3), ((0.0, 1e200, 0.0), 2, 5), ((0.0, 1e200, 0.0), 3, 10),
                                         ((0.0, 0.0, 1e200), 2, 4), ((0.0, 1e100, 1e100), 2, 10),
                                         ((0.0, 1e100, 1e100), 4, 18)])
def test_radial_table_beyond_the_range_is_accepted(coefs, dim, p):
    """A term that overflows stays within the terms of the table: no entry that is exactly zero becomes
    nan by it, and none outside the shape refuses the table. An entry below 1e290 has no intermediate beyond
    the range (a product has the power of the couplings of the term that it adds to); its bound is that of
    sums of some hundreds of rounded terms with moderate cancellation."""
    tab, shape = P.level_table_radial(coefs, dim, 1.0, 1.0, p, 0)
    Q = ov.level_groups([Fraction(c) for c in coefs], dim, p, Fraction(1))
    off = overflowed = 0
    for k, j, ln in shape:
        ref = list(reversed(Q[k][j])) if k < len(Q) else []
        ref = [Fraction(0)] * (ln - len(ref)) + ref
        for got, r in zip(tab[off:off + ln], ref):
            if r == 0:
                assert got == 0.0, (k, j)
            elif abs(r) < 10 ** 290:
                assert abs(got - float(r)) <= 1e-12 * abs(float(r)), (k, j)
            elif abs(r) > 10 ** 309:
                assert not np.isfinite(got), (k, j)
                overflowed += 1
        off += ln
    assert off == tab.size and overflowed > 0


def test_reference_actions_beyond_the_range_are_those_of_the_slices(tmp_path):
    """nan and infinities of the straight-line actions (level 0: the exponent itself, where an infinity in
    place of nan would be an amplitude of 0) are those of a sum of slices; finite ones agree to the rounding of
    32 slices of at most 190 terms: 1e-12 with all terms of one sign, which large couplings give."""
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "check_line")
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "check_line_action.cpp"), "-o", exe], check=True)
    out = np.array(subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split(), dtype=float)
    got, ref = out[0::2], out[1::2]
    fin = np.isfinite(ref)
    assert fin.sum() > 1000 and np.isnan(ref).sum() > 300
    assert np.array_equal(got[~fin], ref[~fin], equal_nan=True)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-12 * np.abs(ref[fin]))


def fma(a, b, c):
    """a b + c with one rounding."""
    a, b, c = float(a), float(b), float(c)
    if not (math.isfinite(a) and math.isfinite(b) and math.isfinite(c)):
        return c if math.isinf(c) and math.isfinite(a) and math.isfinite(b) else a * b + c
    exact = Fraction(a) * Fraction(b) + Fraction(c)
    try:
        return float(exact)
    except OverflowError:
        return math.inf if exact > 0 else -math.inf


def radial_slice(tab, shape, a, b):
    """Action of the slice from a to b from the unscaled table, by Horner in u, z, w^2 in the table's order."""
    u = w = z = 0.0
    for qa, qb in zip(a, b):
        x, h = 0.5 * (qa + qb), 0.5 * (qb - qa)
        u, w, z = fma(x, x, u), fma(x, h, w), fma(h, h, z)
    acc = zs = None
    off = 0
    for n, (k, j, ln) in enumerate(shape):
        v = 0.0
        for e in range(ln):
            v = fma(v, u, tab[off + e]) if e else float(tab[off])
        off += ln
        zs = v if n == 0 or shape[n - 1][1] != j else fma(zs, z, v)
        if n + 1 == len(shape) or shape[n + 1][1] != j:
            acc = zs if acc is None else fma(acc, w * w, zs)
    return acc


@pytest.mark.gpu
@pytest.mark.parametrize("dim,p,T,coefs,a,b", [
    (1, 14, 0.63, (0.0, 6.2e5, 1.1e14), (-4.3e26,), (4.3e26,)),
    (3, 15, 0.026, (0.0, 4.7e13, 1.8e14), (-9e14, -6.7e15, 2.7e16), (2.1e16, 5.9e15, -3.2e16)),
    (3, 11, 0.175, (0.0, 0.56, 7.6e14), (-1.5e32, -7.4e31, 1.5e31), (1.5e32, 7.4e31, -1.5e31)),
    (4, 14, 3.4e6, (0.0, 8.2e3, 9.5e5), (2.5e22, 2.2e22, 4.4e21, -1.1e22), (-2.5e22, -2.2e22, -4.4e21, 1.1e22)),
    (2, 6, 0.5, (0.0, 0.5, 0.2), (0.1, 0.4), (0.9, -0.3))])
def test_radial_level_0_beyond_the_range(dim, p, T, coefs, a, b):
    """The level-0 exponent of the radial route (one slice, no kernel runs at N = 1) where its terms, or only
    their sums over the powers of z, leave the range, and once where nothing does."""
    with P.Context() as ctx:
        res, _ = ctx.amplitude_radial(coefs, dim, 1.0, a, b, T, 1, p, 100, 1)
    with np.errstate(all="ignore"):
        r2 = sum((y - x) ** 2 for x, y in zip(a, b))
        log_k = np.log(np.exp(-r2 / (2.0 * T)) / (2.0 * np.pi * T) ** (0.5 * dim))
        ref = log_k - radial_slice(*P.level_table_radial(coefs, dim, 1.0, T, p, 0), a, b)
    assert np.isclose(res[0].log_amp, ref, rtol=1e-12, atol=1e-12, equal_nan=True)
