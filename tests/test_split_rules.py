"""The rules by which runs are shared out between whole chunks and groups (host code, no device use):
every group once, within the room for group sums, and no more tickets than their groups' work covers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1105_0542_amd", "csrc")
TICKET_NS = 12.4               # of the whole GPU, one address
SLICE_NS = 64 / 550.0          # of the whole GPU: 64 paths of one slice at the cheapest rate, 5.5e11 slices a second


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("split") / "check_split")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "check_split.cpp"), "-o", exe], check=True)
    return [ln.split() for ln in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()]


def test_runs(lines):
    runs = [[int(x) for x in ln[1:]] for ln in lines if ln[0] == "run"]
    assert len(runs) > 1000
    kinds = set()
    for wgs, s, slots, n, groups, chunks, coarse, fine, dealt, grab in runs:
        case = (wgs, s, slots, n)
        assert groups == -(-n // 64) and chunks == -(-n // 4096), case
        assert 0 <= coarse <= chunks and coarse * 64 + fine == max(groups, coarse * 64), case
        assert fine * slots * 24 <= 16 << 20 and grab >= 1, case
        assert (coarse == 0 or slots > 0) and dealt <= fine and (dealt == 0 or coarse == 0), case
        tickets = -(-(fine - dealt) // grab)
        # two rounds of single tickets for the 4 waves of a workgroup may be waited for, not more
        assert tickets * TICKET_NS <= (fine - dealt) * (1 << s) * SLICE_NS + 2 * 4 * wgs * TICKET_NS, case
        kinds.add((coarse > 0, fine > 0, dealt > 0))
    assert kinds >= {(False, True, True), (True, False, False), (True, True, False)}


def test_short_paths_by_chunk_or_by_group(lines):
    """N <= 32: all by chunk from four rounds on and where the last is half full, else all by group."""
    runs = [[int(x) for x in ln[1:]] for ln in lines if ln[0] == "run"]
    runs = [r for r in runs if r[1] <= 5 and r[2] > 0 and r[5] > r[0]]
    seen = set()
    for wgs, s, slots, n, groups, chunks, coarse, fine, dealt, grab in runs:
        assert coarse in (0, chunks), (wgs, s, slots, n)
        if chunks == 513 and wgs == 512:
            assert coarse == 0 and dealt == groups
        if chunks >= 4 * wgs or 8 * chunks // wgs % 8 in (3, 4):
            assert coarse == chunks
        seen.add(coarse == 0)
    assert seen == {True, False}


def test_batch_classes(lines):
    """Whole chunks where there are four or more for every workgroup, groups where there are fewer than
    workgroups; items by ticket are worth their tickets."""
    classes = [[int(x) for x in ln[1:]] for ln in lines if ln[0] == "class"]
    assert len(classes) > 300
    for wgs, s, k, n, chunks, by_group, share, block, items, dealt in classes:
        case = (wgs, s, k, n)
        if chunks >= 4 * wgs:
            assert not by_group, case
        if 2 * chunks < wgs:
            assert by_group, case
        assert block >= 1 and 0 <= dealt <= items, case
        if dealt < items:
            assert block * (1 << s) >= 128 and items - dealt >= min(items, 2 * 4 * wgs), case
        assert dealt == items or block * (1 << s) * SLICE_NS > TICKET_NS, case
    assert {c[5] for c in classes} == {0, 1} and any(c[9] < c[8] for c in classes)


def test_batch_classes_of_long_paths(lines):
    """Fewer than four chunks for every workgroup: by group from 128 slices a group on; full rounds of equal chunks of
    shorter ones by chunk."""
    mixes = [[int(x) for x in ln[1:]] for ln in lines if ln[0] == "mix"]
    assert len(mixes) == 72
    for k, kinds, s, mean, by_group in mixes:
        if k >= 2048:
            assert not by_group, (k, kinds, s)
        elif mean >= 128:
            assert by_group, (k, kinds, s)
        elif kinds == 1 and k % 512 == 0:
            assert not by_group, (k, kinds, s)
