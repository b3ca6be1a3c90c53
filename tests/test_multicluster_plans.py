"""Where multi-cluster Houdayer steps run fused: only with two or more scratch
areas per workgroup (host only)."""
import pytest

from paper_2003_04621_amd import pt


def fused(d, L, NT, **kw):
    return pt.pt_plan_query(d, L, NT, houdayer=True, measure=True, multi=True, **kw)["mode"] == 1


# (dim, L, longest ladder with room for two areas, one with room for one)
@pytest.mark.parametrize("d,L,two,one", [
    (2, 14, 362, 365), (2, 28, 355, 360), (2, 32, 335, 340), (2, 50, 152, 158), (2, 64, 118, 122),
    (2, 64, 118, 127), (3, 10, 292, 296), (3, 12, 157, 160), (3, 16, 115, 119), (3, 18, 61, 67), (3, 22, 8, 11),
    (3, 24, 14, 18), (3, 26, 1, 3), (3, 28, 1, 7)])
def test_one_scratch_area_is_no_plan(d, L, two, one):
    if two >= 2:
        assert fused(d, L, two) and fused(d, L, max(2, two // 2))
    for NT in (two + 1, one):
        assert not fused(d, L, NT), NT


def test_the_extras_take_their_room():
    assert fused(3, 18, 61) and not fused(3, 18, 61, walk=True, modes=True)
    assert fused(3, 18, 56, walk=True, modes=True)
