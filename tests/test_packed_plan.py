"""How the one-launch plan of a packed batch cuts its sequences, on both sides of every line of its rules: segments of the longest sequence, from
the workspace that the batch asks for, and waves of a workgroup of the output pass, from its launch (see launches.py).  CPU only."""
import time

import pytest

from paper_2509_18467_amd import lawcat

import launches as L


def spread(n, lo, hi):
    """n lengths, evenly spread over their logarithm."""
    return [round(lo * (hi / lo) ** (i / (n - 1))) for i in range(n)]


@pytest.fixture(scope="module")
def directory(tmp_path_factory):
    return str(tmp_path_factory.mktemp("launches"))


def plan(directory, d, Hq, Hkv, lengths, room=None):
    """(segments of the longest sequence, waves a workgroup); None if the call is refused"""
    starts = [0]
    for n in lengths:
        starts.append(starts[-1] + n)
    desc = lawcat.make_desc(len(lengths), max(lengths), Hq, Hkv, d)
    need = lawcat.varlen_workspace_bytes(desc, starts, True)
    slot = len(lengths) * Hkv * ((d * d + 2 * d) * 4 + 4)
    assert need % slot == 0
    (status, made), = L.run([L.packed(desc, starts, L.AT, need if room is None else room * slot)], directory)
    return (need // slot or 1, made[-1][3] // 64) if status == 0 else None


# Head dim 64: more workgroups than a round only for segments of 512 tokens and more, and not in the place of uncut sequences
@pytest.mark.parametrize("Hq,Hkv,lengths,segments", [
    (8, 4, spread(12, 403, 985), 8), (64, 32, spread(13, 10, 1933), 3), (16, 16, spread(35, 4, 4317), 1), (16, 8, spread(58, 128, 2923), 3)])
def test_more_than_a_round(directory, Hq, Hkv, lengths, segments):
    assert plan(directory, 64, Hq, Hkv, lengths) == (segments, 4)


# Where uncut sequences are a full round: cut if that leaves two fifths of the longest; not of more than a round, nor where there are more than
# 64, nor where a sequence's workgroups are no multiple of eight
@pytest.mark.parametrize("d,Hq,Hkv,lengths,segments,waves", [
    (64, 32, 8, spread(64, 100, 7743), 3, 4), (64, 16, 16, spread(32, 15, 1500), 3, 4), (64, 16, 16, spread(32, 135, 1947), 1, 4),
    (64, 32, 8, spread(65, 100, 7743), 1, 4), (128, 16, 16, spread(32, 36, 1966), 3, 4), (128, 16, 16, spread(32, 174, 2087), 1, 8), (128, 10, 10, spread(51, 11, 1030), 1, 8),
    (64, 20, 20, spread(25, 20, 1500), 1, 4), (128, 8, 8, spread(64, 10, 1114), 3, 4), (128, 32, 32, spread(17, 35, 474), 1, 8)])
def test_full_round(directory, d, Hq, Hkv, lengths, segments, waves):
    assert plan(directory, d, Hq, Hkv, lengths) == (segments, waves)


# Head dim 64: uncut where the state pass costs more than what it shortens
@pytest.mark.parametrize("Hq,Hkv,lengths,segments", [
    # by 64 tokens: always; in two launches, each of which walks all of it, not
    (8, 8, [93, 97], 1), (64, 8, spread(43, 2, 116), 1), (12, 2, spread(22, 66, 80), 1), (40, 8, spread(15, 36, 86), 2),
    # by 128: by query heads' walks
    (8, 8, [159, 166], 3), (8, 8, spread(8, 150, 185), 3), (8, 8, spread(23, 26, 149), 1), (8, 8, spread(14, 88, 191), 1), (16, 8, spread(4, 22, 148), 3),
    (16, 8, spread(9, 3, 170), 3), (16, 8, spread(13, 29, 158), 1), (32, 8, spread(2, 83, 137), 3), (32, 8, spread(7, 33, 153), 1),
    # by how many sequences are cut where workgroups take four heads
    (32, 8, spread(20, 2, 185), 3), (16, 4, spread(33, 19, 145), 3), (16, 2, spread(78, 10, 250), 2), (32, 8, spread(39, 4, 187), 1),
    # in two launches; long segments
    (20, 4, spread(27, 35, 192), 3), (32, 8, spread(43, 459, 651), 1),
    # in a round more
    (32, 4, spread(64, 70, 448), 1), (128, 16, spread(16, 80, 641), 3), (64, 8, spread(32, 69, 534), 3)])
def test_uncut(directory, Hq, Hkv, lengths, segments):
    assert plan(directory, 64, Hq, Hkv, lengths) == (segments, 4)


# Head dim 128, more uncut workgroups than units: four waves a workgroup where they make the longest walk enough shorter, or have enough work
@pytest.mark.parametrize("Hq,Hkv,lengths,segments,waves", [
    # no more than an eighth more
    (32, 8, [250] * 36, 1, 8), (32, 8, [250] * 37, 1, 4), (32, 8, [250] * 48, 1, 4),
    # cut: one and two heads a group, four, three in two launches; more than a round of them; few sequences of many heads; groups of eight
    (8, 8, spread(47, 28, 1002), 3, 4), (4, 4, spread(88, 22, 288), 1, 8), (8, 8, spread(42, 327, 871), 1, 8), (32, 8, spread(40, 66, 395), 3, 4),
    (32, 8, spread(46, 390, 980), 2, 4), (24, 8, spread(39, 217, 662), 2, 4), (48, 16, spread(27, 9, 342), 1, 8), (8, 8, spread(57, 47, 2893), 4, 4),
    (8, 8, spread(60, 10, 485), 1, 8), (32, 32, spread(13, 213, 1909), 1, 8), (32, 4, spread(44, 8, 1000), 4, 4),
    # uncut: by a unit's share
    (8, 8, spread(70, 4, 760), 1, 8), (40, 8, spread(72, 21, 621), 1, 8), (64, 16, spread(40, 13, 543), 1, 8), (64, 16, [250] * 40, 1, 4),
    (64, 8, spread(36, 39, 345), 1, 4), (16, 8, spread(57, 385, 1812), 1, 4), (8, 8, spread(58, 80, 898), 1, 8), (8, 8, spread(55, 61, 269), 1, 4),
    (16, 8, spread(38, 9, 95), 1, 4), (8, 8, spread(38, 1, 98), 1, 8), (32, 32, spread(13, 96, 571), 1, 8), (32, 32, [571] * 13, 1, 4)])
def test_four_waves(directory, Hq, Hkv, lengths, segments, waves):
    assert plan(directory, 128, Hq, Hkv, lengths) == (segments, waves)


# A workspace too small for the quickest plan takes the one that needs least: its segments of the longest sequence, and its launches
@pytest.mark.parametrize("d,Hq,Hkv,lengths,segments,launches", [
    (128, 32, 8, spread(24, 100, 3269), 3, [(328, 1, 1, 512)] * 2), (128, 8, 8, spread(57, 47, 2893), 0, [(1, 456, 1, 512)]),
    (64, 16, 8, spread(58, 128, 2923), 2, [(664, 1, 1, 256)] * 2)])
def test_least_plan(directory, d, Hq, Hkv, lengths, segments, launches):
    starts = [0]
    for n in lengths:
        starts.append(starts[-1] + n)
    desc = lawcat.make_desc(len(lengths), max(lengths), Hq, Hkv, d)
    slot = len(lengths) * Hkv * ((d * d + 2 * d) * 4 + 4)
    need = lawcat.varlen_workspace_bytes(desc, starts, True)
    assert need > segments * slot
    quick, short, least, null, less = L.run([L.packed(desc, starts, L.AT, room) for room in (need, need - 1, segments * slot)] +
                                            [L.packed(desc, starts, L.NULL, need), L.packed(desc, starts, L.AT, max(0, segments * slot - 1))], directory)
    assert quick[0] == 0 and quick[1] != launches
    assert short == least == (0, launches)
    assert (null == less == (-4, [])) if segments else (null == less == (0, launches))


@pytest.mark.parametrize("d,Hq,Hkv", [(64, 32, 8), (128, 8, 8), (128, 32, 8), (128, 40, 8)])
def test_time(d, Hq, Hkv):
    """A plan does not look at the lengths of a segment one after the other (up to 420 us, 7 by halves): 64 sequences up to 131072 tokens."""
    starts = [0]
    for n in spread(64, 100, 131072):
        starts.append(starts[-1] + n)
    desc = lawcat.make_desc(64, 131072, Hq, Hkv, d)
    best = 1.0
    for _ in range(20):
        t = time.perf_counter()
        lawcat.varlen_workspace_bytes(desc, starts, True)
        best = min(best, time.perf_counter() - t)
    assert best < 1e-4
