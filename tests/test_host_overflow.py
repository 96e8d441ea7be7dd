"""Effective-action tables and reference actions whose terms leave the FP64 range (host code)."""
from fractions import Fraction

import numpy as np
import pytest

import paper_1105_0542_amd as P
from oracle import vector as ov


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
