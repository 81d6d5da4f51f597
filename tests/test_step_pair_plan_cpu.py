"""Which lattices take two steps per launch, from the library's own plan on the host: lattices on which
single steps were faster do not."""
import pytest

from launch_plan import ask

SCALAR, WIDTH1 = 1, 1 << 4


def _line(prec, shape, walls=0, t_mode=0, r_mode=0, flags=0):
    return f"pair {prec} {flags} {walls} {t_mode + 4 * r_mode} {shape[0]} {shape[1]} {shape[2]}"


# FP64 whole rows: single steps were faster (or no slower) with walls or a source at these
@pytest.mark.parametrize("shape,walls,t_mode,r_mode", [((112, 112, 112), 1, 2, 2), ((112, 112, 112), 1, 2, 0),
                                                       ((112, 112, 112), 0, 0, 2), ((120, 120, 120), 1, 2, 2),
                                                       ((88, 88, 88), 1, 2, 2), ((80, 80, 80), 1, 2, 2)])
def test_whole_rows_with_walls_and_sources_stay_single(shape, walls, t_mode, r_mode):
    assert ask([_line("f64", shape, walls, t_mode, r_mode)])[0][0] == 0


def test_other_routes_stay_single():
    big = (128, 128, 128)
    assert ask([_line("f32", big)])[0][0] == 1
    assert [p[0] for p in ask([_line("f32", big, flags=SCALAR), _line("f32", big, flags=WIDTH1),
                               _line("f32", (64, 64, 64)), _line("f64", (48, 48, 48))])] == [0, 0, 0, 0]
    assert ask([_line("f32", big)], 27)[0][0] == 0
