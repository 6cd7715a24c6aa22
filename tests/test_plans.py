"""Single steps or passes: the choice against measured times (MI355X, us per step), where
one side was faster by 5 % or more."""
import pytest

from plans import planes_per_segment, tile

X, Y, Z, ALL = (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1)


@pytest.mark.parametrize("shape,bc", [
    ((64, 64, 64), X), ((64, 64, 64), ALL),          # 13.8 against 15.5
    ((128, 128, 128), X), ((128, 128, 128), ALL),    # 59 against 76
    ((160, 160, 160), X), ((192, 192, 192), X),      # 124 against 133, 212 against 223
    ((200, 100, 150), X), ((200, 100, 150), ALL),    # 91 against 103
    ((40, 3, 90), Z),                                # 6.4 against 6.9
])
def test_walled_d3v19_boxes_that_keep_single_steps(shape, bc):
    assert planes_per_segment(shape, bc) == 0


@pytest.mark.parametrize("shape,bc", [
    ((48, 48, 48), X), ((80, 80, 80), X), ((100, 100, 100), X), ((88, 36, 236), ALL), ((24, 24, 256), X),
    ((250, 30, 30), X), ((62, 140, 140), ALL),
    ((80, 80, 80), Y), ((100, 100, 100), Y), ((192, 192, 192), Y), ((160, 160, 160), Y), ((256, 256, 256), Y), ((24, 24, 256), Y),
    ((64, 64, 64), Z), ((125, 16, 50), Z), ((100, 100, 100), Z), ((160, 160, 160), Z), ((200, 100, 150), Z), ((256, 256, 256), Z),
])
def test_walled_d3v19_boxes_that_take_passes(shape, bc):
    assert planes_per_segment(shape, bc) > 0


@pytest.mark.parametrize("shape", [(30, 30, 30), (64, 64, 64), (128, 128, 128), (200, 100, 150), (256, 256, 256)])
@pytest.mark.parametrize("bc", [X, Y, Z, ALL])
def test_walled_d3v19_boxes_in_float64_take_passes(shape, bc):
    assert planes_per_segment(shape, bc, fp64=True) > 0


@pytest.mark.parametrize("shape,fp64,porous", [
    ((200, 200), False, False), ((256, 256), False, False), ((300, 300), False, False),  # 5.1 : 6.2, 5.3 : 6.2, 6.3 : 7.7
    ((360, 360), False, False), ((256, 256), False, True), ((180, 180), True, False), ((300, 300), True, False),
    ((230, 230), True, True),
])
def test_single_steps_where_a_tile_of_one_step_takes_longer(shape, fp64, porous):
    p = tile(shape, fp64, porous=porous)
    assert p.h > 1 and not p.one


@pytest.mark.parametrize("shape,fp64,porous", [
    ((80, 80), False, False), ((512, 64), False, False), ((2048, 32), False, False), ((8192, 8), False, False),
    ((16, 1024), True, False), ((700, 150), True, True), ((1000, 60), True, False), ((160, 160), False, True),
])
def test_tiles_of_one_step_where_they_are_faster(shape, fp64, porous):
    assert tile(shape, fp64, porous=porous).one
