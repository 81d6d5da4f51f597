"""The benchmark's bytes per step where a launch takes two steps: populations once per launch,
coefficients in every step."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402
from paper_2605_01774_amd import inputs as I  # noqa: E402


def test_bytes_that_a_step_moves():
    decay = I.fourier_decay(n=8, steps=1)
    assert bench.moved_bytes_per_lup("f32", decay) == 152
    assert bench.moved_bytes_per_lup("f32", decay, per_launch=2) == 76
    porous = I.porous_spheres(n=8, steps=1)
    assert bench.moved_bytes_per_lup("f64", porous, per_launch=2) == 152 + 6 * 8
    assert bench.moved_bytes_per_lup("f64", porous, phases=True, per_launch=2) == 152 + 1
    field = I.variable_tensor_source(n=8, steps=1)
    assert bench.moved_bytes_per_lup("f64", field) == bench.bytes_per_lup("f64", field)
