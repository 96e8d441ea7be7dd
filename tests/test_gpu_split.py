"""How a run's paths are shared out (whole chunks by a workgroup, groups of 64 paths by a wave, dealt or
by ticket) does not show in the canonical chunk sums: every split gives the same bits."""
import numpy as np
import pytest

import paper_1105_0542_amd as P

pytestmark = pytest.mark.gpu
CHUNK = 4096
FINE_BYTES = 16 << 20          # group sums a run keeps (24 bytes per group and level): beyond, whole chunks


@pytest.fixture(scope="module")
def ctx():
    with P.Context() as c:
        yield c


def run(ctx, route, s, n, flags):
    if route == "radial":
        ctx.amplitude_radial([0.0, 0.5, 0.2], 2, 1.0, (0.0, 0.1), (0.6, 0.2), 0.8, 1 << s, 1, n, 5, 3, flags)
    elif route == "noalloc":
        ctx.amplitude_noalloc(P.quartic(1.0, 2.0), 1.0, 0.0, 0.7, 0.8, 1 << s, 1, n, 5, 3, flags)
    else:
        ctx.amplitude(P.quartic(1.0, 2.0), 1.0, 0.0, 0.7, 0.8, 1 << s, 1, n, 5, 3, flags)


def chunks(ctx, level, picks):
    return np.stack([ctx.last_partials(level, c, 1)[0][0] for c in picks])


@pytest.mark.parametrize("route,s,flags", [("quartic", 4, 0), ("quartic", 6, 0), ("radial", 3, 0),
                                           ("noalloc", 4, P.FLAG_HIERARCHY)])
def test_whole_chunks_and_groups_give_the_same_sums(ctx, route, s, flags):
    slots = s + 1 if flags else 1
    fit = FINE_BYTES // (slots * 64 * 24)
    if route == "noalloc":     # chunk records that leave no room for group sums: every chunk whole
        n = (16_513_792 // (32 * slots)) * CHUNK - 1000
    else:                      # forty whole chunks, the rest by group
        n = (fit + 40) * CHUNK - 1000
    total = -(-n // CHUNK)
    picks = [0, 1, 17, 38, 39, 40, 41, 60]
    run(ctx, route, s, n, flags)
    level = s if not flags else 2
    whole = chunks(ctx, level, picks)
    assert ctx.last_partials(level, total - 1, 1)[0][0][0] == n - (total - 1) * CHUNK
    # a run of 64 chunks goes by group throughout
    run(ctx, "quartic" if route == "noalloc" else route, s, 64 * CHUNK, flags)
    assert np.array_equal(whole, chunks(ctx, level, picks))


@pytest.mark.parametrize("s", [3, 4, 6, 8])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 4095, 4096, 4097, 131_072 + 65, 600_001])
def test_ragged_runs_agree_with_their_paths(ctx, s, n):
    """Chunk sums against the per-path actions of the same run: d = expm1(S_ref - S) summed in FP64. The
    bound is that of a sum of 4096 terms in any order, 4096 2^-53 sum|d|, and of expm1 to 4 ulp."""
    run(ctx, "quartic", s, n, P.FLAG_HIERARCHY)
    total = -(-n // CHUNK)
    for c in sorted({0, total // 2, total - 1}):
        rec, _, tc, shift = ctx.last_partials(s, c, 1)
        assert tc == total
        k = min(CHUNK, n - c * CHUNK)
        S = ctx.path_actions(P.quartic(1.0, 2.0), 1.0, 0.0, 0.7, 0.8, 1 << s, 1, 5, 3, P.FLAG_HIERARCHY, c * CHUNK, k)
        d = np.expm1(shift - S[:, s])
        tol = (4096 + 8) * 2.0 ** -53 * np.abs(d).sum()
        assert rec[0][0] == k and rec[0][3] == 0
        assert abs(rec[0][1] - d.sum()) <= tol
        assert abs(rec[0][2] - (d * d).sum()) <= 2 * tol * max(1.0, np.abs(d).max())


@pytest.mark.parametrize("big,flags", [(200_000_000, 0), (40_000_001, P.FLAG_HIERARCHY), (70_001, 0), (70_001, P.FLAG_HIERARCHY)])
def test_batch_items_by_chunk_and_by_group_equal_single_calls(ctx, big, flags):
    """200e6 paths have 3.1e6 groups, beyond the 2.8e6 whose sums a batch keeps (whole chunks); 40e6 with
    five levels likewise; 70,001 go by group. Ragged and short tasks of other N beside them."""
    rows = [(0, 1.0, 0.0, 0.7, 0.8, 16, 1, big, 3), (0, 1.0, 0.1, 0.5, 0.8, 32, 1, 4097, 4),
            (0, 1.0, 0.2, 0.5, 0.8, 128, 1, 65, 5), (0, 1.0, 0.2, 0.4, 0.8, 64, 2, 2, 6), (0, 1.0, 0.2, 0.4, 0.8, 16, 2, 63, 7)]
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
