"""Reference actions of the straight line (the shift of the chunk sums) formed on the device by the general
mode and the component route: against the oracle's slice actions summed along the line, and the same
bits for level n whatever the run's N (the levels split into parts from n = 9 on). Tolerance: the parity
bound of the slice actions, 1e-12 of max(1, sum of absolute slice actions)."""
import numpy as np
import pytest

import paper_1105_0542_amd as P
from oracle import general as og
from oracle import vector as ov

pytestmark = pytest.mark.gpu
H = P.FLAG_HIERARCHY
SECH, GAUSS, POLY = ((0.5, 0.8),), ((1.5, 1.0),), (0.1, 0.2, 0.5, 0.0, 0.05)
TERMS = [(0.5, (2, 0)), (0.7, (0, 2)), (0.1, (4, 0)), (0.6, (2, 2)), (0.3, (1, 0)), (0.2, (1, 1))]


@pytest.fixture(scope="module")
def ctx():
    with P.Context() as c:
        yield c


def shifts(ctx, s):
    return [ctx.last_partials(n, 0, 1)[3] for n in range(1, s + 1)]


@pytest.mark.parametrize("p,s", [(3, 1), (4, 9), (8, 8), (8, 15), (12, 10), (13, 3)])
def test_general_mode_lines(ctx, p, s):
    a, b, T = -0.4, 0.9, 0.8

    def run(s):
        ctx.amplitude_general(1.0, a, b, T, 1 << s, p, 128, 1, 0, H, poly=POLY, sech2=SECH, gauss=GAUSS)
        return shifts(ctx, s)

    got = run(s)
    dfun = og.derivative_functions(p, POLY, SECH, GAUSS, 1.0)
    for n in {1, min(2, s), s}:
        q = a + (b - a) * np.arange((1 << n) + 1) / (1 << n)
        w = og.eps_W(p, T / (1 << n), dfun, 0.5 * (q[1:] + q[:-1]), 0.5 * (q[1:] - q[:-1]))
        assert abs(got[n - 1] - w.sum()) <= 1e-12 * max(1.0, np.abs(w).sum()), n
    if s > 1:
        assert run(s - 1) == got[:-1]


@pytest.mark.parametrize("p,s", [(4, 1), (5, 8), (3, 14)])
def test_component_route_lines(ctx, p, s):
    a, b, T = (0.1, -0.2), (0.8, 0.5), 0.7

    def run(s):
        ctx.amplitude_poly(TERMS, 2, 1.0, a, b, T, 1 << s, p, 128, 1, 0, H)
        return shifts(ctx, s)

    got = run(s)
    tabs = ov.component_tables(ov.terms_to_components(TERMS, 2), 2, p, T, s)
    for n in {1, s}:
        k = np.arange((1 << n) + 1)[:, None] / (1 << n)
        q = np.array(a) + (np.array(b) - np.array(a)) * k
        x, xb = 0.5 * (q[1:] + q[:-1]), 0.5 * (q[1:] - q[:-1])
        w, scale = ov.component_eps_W(tabs[n], x, xb), ov.component_eps_W_abs(tabs[n], x, xb)
        assert abs(got[n - 1] - w.sum()) <= 1e-12 * max(1.0, scale.sum()), n
    if s > 1:
        assert run(s - 1) == got[:-1]
