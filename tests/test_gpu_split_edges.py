"""Runs and batches at the edges of the rules that share them out (pimc_split.hpp; 512 workgroups resident):
the kernel of whole chunks alone, whole chunks with groups behind them, groups alone."""
import numpy as np
import pytest

import paper_1105_0542_amd as P

pytestmark = pytest.mark.gpu
CHUNK = 4096


@pytest.fixture(scope="module")
def ctx():
    with P.Context() as c:
        yield c


def run(ctx, route, s, n, flags):
    if route == "quartic":
        ctx.amplitude(P.quartic(1.0, 2.0), 1.0, 0.0, 0.7, 0.8, 1 << s, 2, n, 5, 3, flags)
    elif route == "fp32":
        ctx.amplitude(P.quartic(1.0, 2.0), 1.0, 0.0, 0.7, 0.8, 1 << s, 2, n, 5, 3, flags | P.FLAG_FP32_POLY)
    elif route == "odd":
        ctx.amplitude([0.0, 0.3, 0.5, 0.1, 0.2], 1.0, 0.0, 0.7, 0.3, 1 << s, 2, n, 5, 3, flags)
    elif route == "mpt":
        ctx.amplitude_mpt(1.0, 1.0, 1.0, 0.0, 0.5, 0.5, 1 << s, 2, n, 5, 3, flags)
    elif route == "general":
        ctx.amplitude_general(1.0, 0.1, 0.9, 0.4, 1 << s, 1, n, 5, 3, flags, poly=[0, 0, 0.5], gauss=[(1.0, 0.8)])
    elif route == "radial":
        ctx.amplitude_radial([0.0, 0.5, 0.2], 2, 1.0, (0.0, 0.1), (0.6, 0.2), 0.8, 1 << s, 1, n, 5, 3, flags)
    else:
        ctx.amplitude_poly([(0.5, (2, 0)), (0.4, (0, 2)), (0.2, (1, 1))], 2, 1.0, (0.0, 0.1), (0.6, 0.2), 0.8, 1 << s, 1, n,
                           5, 3, flags)


@pytest.mark.parametrize("chunks", [512, 513, 717, 1301, 1537])
@pytest.mark.parametrize("route,s,flags", [("quartic", 3, 0), ("quartic", 5, P.FLAG_HIERARCHY), ("quartic", 6, P.FLAG_HIERARCHY),
                                           ("fp32", 5, 0), ("odd", 4, 0), ("mpt", 6, 0), ("general", 6, 0), ("radial", 6, 0),
                                           ("poly", 6, 0)])
def test_chunk_sums_do_not_depend_on_the_share(ctx, route, s, flags, chunks):
    """Chunk sums against a run of 48 chunks (groups alone). The ragged last one of the quartic route against the
    actions of its paths: the bound is that of a sum of 4096 terms in any order and of expm1 to 4 ulp."""
    n = chunks * CHUNK - 1001
    run(ctx, route, s, n, flags)
    level = s if not flags else s - 1
    got = ctx.last_partials(level, 0, chunks)[0]
    shift = ctx.last_partials(level, 0, 1)[3]
    assert np.all(got[:-1, 0] == CHUNK) and got[-1, 0] == CHUNK - 1001 and np.all(got[:, 3] == 0)
    assert np.all(np.isfinite(got)) and np.all(got[:, 2] > 0)
    run(ctx, route, s, 48 * CHUNK, flags)
    assert np.array_equal(got[:48], ctx.last_partials(level, 0, 48)[0])
    if route == "quartic":
        S = ctx.path_actions(P.quartic(1.0, 2.0), 1.0, 0.0, 0.7, 0.8, 1 << s, 2, 5, 3, P.FLAG_HIERARCHY, (chunks - 1) * CHUNK,
                             CHUNK - 1001)
        d = np.expm1(shift - S[:, level])
        tol = (4096 + 8) * 2.0 ** -53 * np.abs(d).sum()
        assert abs(got[-1, 1] - d.sum()) <= tol and abs(got[-1, 2] - (d * d).sum()) <= 2 * tol * max(1.0, np.abs(d).max())


@pytest.mark.parametrize("flags", [0, P.FLAG_HIERARCHY])
@pytest.mark.parametrize("big", [128 * CHUNK, 128 * CHUNK + 1, 200 * CHUNK - 63, 449 * CHUNK + 65])
def test_batch_segments_of_many_chunks_equal_single_calls(ctx, big, flags):
    """Up to 128 chunks a segment is reduced by one workgroup, beyond its records are formed in pieces of 64."""
    rows = [(0, 1.0, 0.0, 0.7, 0.8, 16, 2, big, 3), (0, 1.0, 0.1, 0.5, 0.8, 16, 2, 4097, 4), (0, 1.0, 0.2, 0.5, 0.8, 64, 3, 70_001, 5)]
    bt = P.Batch(ctx, [P.quartic(1.0, 2.0)], rows, 5, flags)
    res, _, _ = bt.run()
    again, _, _ = bt.run()
    bt.close()
    assert res.tobytes() == again.tobytes()
    for i, (_, m, a, b, T, N, p, n, stream) in enumerate(rows):
        one, _ = ctx.amplitude(P.quartic(1.0, 2.0), m, a, b, T, N, p, n, 5, stream, flags)
        for level, r in enumerate(one):
            got = res[i, level]
            assert (got["amp"], got["err"], got["n"]) == (r.amp, r.err, r.n), (i, level)
