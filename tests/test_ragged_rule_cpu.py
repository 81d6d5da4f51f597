"""Where the row-vector kernel's form for ragged rows is taken: at shapes on both sides of its lines,
from the library's own rule on the host."""
import pytest

from launch_plan import ask

REST, SR = 2, 4

# (flags, velocity mode, tensor mode, nx, ny, nz) -> wavefronts of a row, 0: not taken
TAKEN = [(REST | SR, 0, 0, 200, 150, 100, 2), (REST, 0, 0, 200, 150, 100, 2), (SR, 0, 2, 342, 80, 129, 3),
         (REST | SR, 0, 2, 126, 78, 79, 1), (REST | SR, 0, 0, 510, 40, 39, 4)]
REFUSED = [(REST | SR, 0, 0, 200, 27, 28), (REST | SR, 0, 2, 118, 8, 8), (REST | SR, 0, 0, 300, 23, 22),   # too few
           (REST | SR, 0, 0, 96, 205, 203), (REST | SR, 0, 0, 186, 150, 140),                              # too few lanes
           (REST | SR, 0, 0, 201, 150, 100),                                                               # odd
           (0, 0, 0, 200, 150, 100), (REST | SR, 1, 0, 200, 150, 100), (REST | SR, 0, 1, 200, 150, 100)]   # other kernels


@pytest.mark.parametrize("q", [19, 27])
def test_ragged_form_is_taken_where_it_was_faster(q):
    lines = [f"vec b16 {' '.join(str(v) for v in c[:6])}" for c in TAKEN + REFUSED]
    for c, (V, W, waves) in zip(TAKEN + REFUSED, ask(lines, q)):
        want = c[6] if len(c) > 6 else 0
        assert (V, W, waves) == (2 if want else 0, 0, want), c


def test_rows_of_many_wavefronts():
    line = ["vec b16 6 0 0 1000 64 63"]
    assert ask(line, 19)[0] == [2, 0, 8] and ask(line, 27)[0] == [0, 0, 0]
    assert ask(["vec b16 6 0 0 1000 23 22"], 19)[0] == [0, 0, 0]


@pytest.mark.parametrize("q", [19, 27])
def test_gpu_test_shapes_take_the_form(q):
    import test_gpu_ragged_form as t
    lines = [f"vec b16 {flags} 0 {mode} {nx} {ny} {nz}" for nx, ny, nz in t.SHAPES + (t.LONG if q == 19 else [])
             for flags in (REST, SR, REST | SR) for mode in (0, 2)]
    for line, (V, W, waves) in zip(lines, ask(lines, q)):
        assert (V, W) == (2, 0) and waves > 0, line
