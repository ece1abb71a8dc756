"""How the one-launch plan of a packed batch cuts its sequences, on both sides of every line of its rules: segments of the longest sequence, from
the workspace that the batch asks for, and waves of a workgroup of the output pass, from its launch (see launches.py).  CPU only."""
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
    (20, 4, spread(27, 35, 192), 3), (32, 8, spread(43, 459, 651), 1)])
def test_uncut(directory, Hq, Hkv, lengths, segments):
    assert plan(directory, 64, Hq, Hkv, lengths) == (segments, 4)
