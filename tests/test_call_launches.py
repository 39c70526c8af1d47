"""The launches that a call reports for its frame size are those of the tables
it chooses (no table given) or was given."""
import pytest

import paper_1703_02563_amd as ff


@pytest.mark.parametrize("W,H,level,iters,expect", [
    (160, 120, 0, 6, 2),    # 8x8 tiles, a halo of 6, three steps per launch
    (1024, 436, 0, 6, 3),   # 32x12 tiles, a halo of 2: two steps
    (1024, 436, 4, 6, 2),   # 4x4 tiles, a halo of 4, three steps
    (64, 48, 6, 6, 1),      # one cell: as many steps as a halo of 6 takes
    (64, 48, 6, 12, 2), (65, 48, 6, 6, 2), (64, 65, 6, 6, 2), (33, 20, 6, 4, 1), (16, 9, 4, 6, 1),
])
def test_launches_of_a_call_without_a_table(W, H, level, iters, expect):
    assert ff.level_launches(ff.Params(iters=iters), level, size=(W, H)) == expect


def test_launches_of_a_call_with_a_table():
    t = ff.default_tuning().replace(variant=[3] * 7, passes=[2] * 7)
    p = ff.Params(iters=6, tuning=t)
    assert all(ff.level_launches(p, lv, size=(160, 120)) == ff.level_launches(p, lv) == 3 for lv in range(7))
    assert ff.level_launches(ff.Params(iters=6), 0, cost_kind=1, size=(160, 120)) == 6  # float features: a step each


@pytest.mark.parametrize("kw", [dict(size=(0, 5)), dict(size=(5, 40000)), dict(size=(5, 5), ndir=3),
                                dict(size=(5, 5), cost_kind=2)])
def test_out_of_range(kw):
    assert ff.level_launches(ff.Params(iters=6), 0, **kw) == -1
