"""The batch autotuner's cache file."""
import pytest

import paper_1105_0542_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with P.Context() as c:
        yield c


def test_autotune_cache_tells_what_an_item_is(ctx, tmp_path):
    """The choice counts items, groups in a batch of few chunks and whole chunks in one of many, so the two do
    not share an entry; and an entry that does not say which (the key without it) is not taken over."""
    path = tmp_path / "tune.txt"
    rows = {"few": [(0, 1.0, 0.0, 0.7, 0.8, 16, 1, 70_001, 3)], "many": [(0, 1.0, 0.0, 0.7, 0.8, 16, 1, 12_000_000, 3)]}
    for n in rows:
        bt = P.Batch(ctx, [P.quartic(1.0, 2.0)], rows[n], seed=1)
        bt.autotune(str(path))
        bt.close()
    lines = path.read_text().split("\n")[:-1]
    assert len(lines) == 2 and lines[0].split()[0] != lines[1].split()[0]
    old = lines[0].replace("groups", "").replace("chunks", "").split()
    path.write_text(" ".join([old[0], "8", "64"] + old[3:]) + "\n")
    bt = P.Batch(ctx, [P.quartic(1.0, 2.0)], rows["few"], seed=1)
    choice = bt.autotune(str(path))
    bt.close()
    assert choice != (8, 64) and len(path.read_text().split("\n")[:-1]) == 2
