"""Which lattices take two steps per launch, from the library's own plan on the host: those of the GPU
tests do, on tiles that cover them; and lattices on which single steps were faster do not."""
import pytest

from launch_plan import ask

SCALAR, WIDTH1 = 1, 1 << 4


def _line(prec, shape, walls=0, t_mode=0, r_mode=0, flags=0):
    return f"pair {prec} {flags} {walls} {t_mode + 4 * r_mode} {shape[0]} {shape[1]} {shape[2]}"


def test_gpu_test_lattices_take_two_steps():
    import test_gpu_step_capture as capture
    import test_gpu_step_pairs_wide as t
    lines = [_line(p, s, walls, t.T_MODE[te], t.R_MODE[so]) for p, s, te, so in t.CASES for walls in (0, 1)]
    lines += [_line(p, s, r_mode=1) for p, s in capture.CASES[:2]]
    lines += [_line(p, s, walls, t.T_MODE[te]) for walls in (0, 1)
              for p, s, te in [("f64", (240, 163, 160), "field"), ("f64", (64, 211, 203), "uniform"),
                               ("f32", (320, 157, 160), "field"), ("f32", (96, 96, 99), "table")]]
    for line, plan in zip(lines, ask(lines)):
        assert plan[0] == 1, line
        nx, ny, nz = (int(v) for v in line.split()[-3:])
        _, bx, by, ln, tx, ty, tz = plan
        assert (tx - 1) * bx < nx <= tx * bx and (ty - 1) * by < ny <= ty * by and (tz - 1) * ln < nz <= tz * ln, line
        halo = 0 if tx == 1 else 2
        assert (bx + halo) * (by + 2) <= (1024 if " f32 " in line else 512), line


def test_both_kinds_of_tile_are_tested():
    import test_gpu_step_pairs_wide as t
    lines = [_line(p, s, 0, t.T_MODE[te], t.R_MODE[so]) for p, s, te, so in t.CASES]
    seen = {(c[0], c[2], plan[4] > 1) for c, plan in zip(t.CASES, ask(lines))}
    for prec in ("f32", "f64"):
        for tensor in ("uniform", "table", "field") if prec == "f32" else ("uniform", "field"):
            assert (prec, tensor, False) in seen
        assert (prec, "field", True) in seen


# FP64 whole rows: single steps were faster (or no slower) with walls or a source at these
@pytest.mark.parametrize("shape,walls,t_mode,r_mode", [((112, 112, 112), 1, 2, 2), ((112, 112, 112), 1, 2, 0),
                                                       ((112, 112, 112), 0, 0, 2), ((120, 120, 120), 1, 2, 2),
                                                       ((88, 88, 88), 1, 2, 2)])
def test_whole_rows_with_walls_and_sources_stay_single(shape, walls, t_mode, r_mode):
    assert ask([_line("f64", shape, walls, t_mode, r_mode)])[0][0] == 0


def test_other_routes_stay_single():
    big = (128, 128, 128)
    assert ask([_line("f32", big)])[0][0] == 1
    assert [p[0] for p in ask([_line("f32", big, flags=SCALAR), _line("f32", big, flags=WIDTH1),
                               _line("f32", (64, 64, 64)), _line("f64", (48, 48, 48))])] == [0, 0, 0, 0]
    assert ask([_line("f32", big)], 27)[0][0] == 0


# and two steps were faster on tiles of more rows
@pytest.mark.parametrize("shape", [(33, 175, 173), (20, 225, 222), (66, 123, 123), (84, 109, 109)])
def test_tiles_of_more_rows_take_two_steps_between_walls(shape):
    assert ask([_line("f64", shape, 1, 2, 0)])[0][0] == 1
