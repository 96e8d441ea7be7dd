"""The component evaluator's subtrees: a run of 2^s slices is one subtree of s levels up to the deepest
(5, 6 or 7 levels by dimension) and several subtrees of that depth beyond, each depth a kernel of its own.
Level n of a run is formed from the same path points, slices and group sums as a run of 2^n slices, so the
results agree bit for bit (the tests against the oracle are in test_gpu_vector_poly)."""
import numpy as np
import pytest

import paper_1105_0542_amd as P

pytestmark = pytest.mark.gpu

TERMS = {
    1: [(0.3, (1,)), (0.5, (2,)), (0.1, (4,))],
    2: [(0.5, (2, 0)), (0.7, (0, 2)), (0.2, (1, 1)), (0.1, (2, 2)), (0.05, (3, 0))],
    3: [(0.5, (2, 0, 0)), (0.4, (0, 2, 0)), (0.6, (0, 0, 2)), (0.1, (1, 1, 1)), (0.1, (0, 2, 2))],
    4: [(0.5, (2, 0, 0, 0)), (0.4, (0, 2, 0, 0)), (0.6, (0, 0, 2, 0)), (0.5, (0, 0, 0, 2)), (0.1, (1, 1, 0, 1))],
}


@pytest.mark.parametrize("d,p", [(1, 6), (2, 5), (3, 3), (4, 2)])
def test_levels_do_not_depend_on_the_subtree(d, p):
    a, b, n, T, s_max = [0.1] * d, [0.4] * d, 200, 0.8, 8
    with P.Context() as ctx:
        deep = ctx.path_actions_poly(TERMS[d], d, 1.5, a, b, T, 1 << s_max, p, 7, 2, P.FLAG_HIERARCHY, 0, n)
        full = ctx.amplitude_poly(TERMS[d], d, 1.5, a, b, T, 1 << s_max, p, n, 7, 2, P.FLAG_HIERARCHY)[0]
        alone = ctx.amplitude_poly(TERMS[d], d, 1.5, a, b, T, 1 << s_max, p, n, 7, 2)[0]
        assert alone[-1].amp == full[-1].amp
        for s in range(1, s_max):
            S = ctx.path_actions_poly(TERMS[d], d, 1.5, a, b, T, 1 << s, p, 7, 2, P.FLAG_HIERARCHY, 0, n)
            r = ctx.amplitude_poly(TERMS[d], d, 1.5, a, b, T, 1 << s, p, n, 7, 2, P.FLAG_HIERARCHY)[0]
            assert np.all(np.isfinite(S))
            assert np.array_equal(S, deep[:, :s + 1]), (d, s)
            assert [q.amp for q in r] == [q.amp for q in full[:s + 1]], (d, s)
