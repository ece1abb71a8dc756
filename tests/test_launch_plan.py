"""Which launches a prefill makes of the workspace that it is given, read from the launches themselves (see launches.py).  CPU only."""
import pytest

from paper_2509_18467_amd import lawcat

import launches as L

SLOT = (128 * 128 + 2 * 128) * 4 + 4


@pytest.fixture(scope="module")
def directory(tmp_path_factory):
    return str(tmp_path_factory.mktemp("launches"))


def test_no_workspace_has_no_room(directory):
    """Head dim 128, more uncut workgroups than compute units: the quickest plan cuts sequences, and one that needs no workspace is taken as
    well.  Without a pointer it is the one that runs, whatever size is passed beside it."""
    d = lawcat.make_desc(40, 700, 32, 8, 128)
    room = lawcat.workspace_bytes(d, lawcat.CALL_LAYER_PREFILL)
    assert room == 40 * 8 * 2 * SLOT
    one = lawcat.make_desc(1, 128 * 300, 64, 1, 128)
    quick, bare, null, sized, missing = L.run([L.prefill(d, L.AT, room), L.prefill(d, L.AT, 0), L.prefill(d, L.NULL, 0), L.prefill(d, L.NULL, room),
                                               L.prefill(one, L.NULL, 1 << 30)], directory)
    assert quick == (0, [(1, 320, 1, 512), (2, 320, 1, 256)])     # state pass, output pass with four waves
    assert bare == null == sized == (0, [(1, 320, 1, 512)])       # one segment each, eight waves
    assert missing == (-4, [])


@pytest.mark.parametrize("d,Hq,Hkv,B,T", [
    # head dim 128: the four-wave form's slots, more than the limit of the least plan; the same within it; the most slots there are; eight waves
    (128, 32, 8, 1, 18000), (128, 32, 8, 1, 131072), (128, 32, 4, 8, 1025), (128, 4, 1, 511, 700), (128, 32, 8, 1, 16384), (64, 32, 8, 1, 32768)])
def test_static_scratch_has_room_for_the_same_plan(directory, d, Hq, Hkv, B, T):
    desc = lawcat.make_desc(B, T, Hq, Hkv, d)
    static, prefill = L.run([L.static(desc), L.prefill(desc, L.AT, lawcat.workspace_bytes(desc, lawcat.CALL_LAYER_PREFILL))], directory)
    assert static == prefill and static[0] == 0 and len(static[1]) >= 2


@pytest.mark.parametrize("heads,d,B,T,W,one", [
    # as many workgroups as compute units with three taps or four, twice as many with fewer
    (64, 128, 1, 128, 4, True), (65, 128, 1, 128, 4, False), (128, 64, 2, 33, 3, True), (96, 128, 4, 30, 3, False),
    (128, 128, 4, 20, 2, True), (129, 128, 1, 128, 2, False), (128, 128, 3, 50, 1, True), (192, 128, 3, 50, 1, False)])
def test_conv_adjoint_in_one_launch(directory, heads, d, B, T, W, one):
    desc = lawcat.make_desc(B, T, heads, heads, d, conv_width=W)
    (status, launches), = L.run([L.conv_adjoint(desc, heads, L.AT, 1 << 30)], directory)
    assert status == 0 and len(launches) == (1 if one else 2)
    assert not one or launches == [(heads * d // 32, 1, 1, 512)]
