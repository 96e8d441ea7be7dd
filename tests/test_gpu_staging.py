"""Host memory that a context keeps page-locked for its uploads."""
import itertools

import numpy as np
import pytest

import paper_1105_0542_amd as P

pytestmark = pytest.mark.gpu


def mapped():
    """Bytes of device and of page-locked host memory in this process (both are mappings of the GPU's file)."""
    ends = [ln.split()[0].split("-") for ln in open("/proc/self/maps") if "/dev/dri/render" in ln]
    return sum(int(b, 16) - int(a, 16) for a, b in ends)


def test_large_tables_are_not_kept_page_locked():
    """A component table of 3.6 MB and more is on the device once, and not a second time in page-locked memory
    (beyond the first MiB); before and after it the same results."""
    terms = [e for e in itertools.product(range(5), repeat=4) if 0 < sum(e) <= 4]
    terms = [(0.01 + 0.001 * i, e) for i, e in enumerate(terms)]
    a, b, T, s = [0.0] * 4, [0.1] * 4, 0.05, 11
    bytes_up = 8 * (s + 1) * P.level_table_poly(terms, 4, 1.0, T, 11, 0)[0].size
    assert bytes_up > 3_500_000

    def actions(ctx, p):
        return ctx.path_actions_poly(terms, 4, 1.0, a, b, T, 1 << s, p, 1, 0, 0, 0, 64)

    with P.Context() as ctx:
        small = actions(ctx, 2)                  # the same kernel: its scratch memory is there from now on
        before = mapped()
        large = actions(ctx, 11)
        assert mapped() - before < 1.5 * bytes_up + (1 << 20)
        assert np.array_equal(small, actions(ctx, 2)) and np.array_equal(large, actions(ctx, 11))
        assert np.all(np.isfinite(large)) and np.allclose(large[:, s], small[:, s], rtol=1e-3)
