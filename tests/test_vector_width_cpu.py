"""Which step kernel a row of 64 V W nodes takes, from the library's own rule on the host: the faster
measured one at shapes on both sides of the rule's lines, and at lattices of few rows."""
import pytest

from launch_plan import ask

# (D3Q, form, flags, velocity mode, tensor mode, nx, ny, nz) -> nodes per lane (0: one per thread),
# wavefronts. Times in us per step of the alternatives
CHOICES = [
    (19, "b16", 0, 1, 1, 384, 103, 101, 2, 3),    # V1 73, V2 67
    (19, "b16", 6, 1, 1, 384, 103, 101, 2, 3),    # V1 88, V2 73
    (27, "b16", 6, 1, 1, 384, 103, 101, 2, 3),    # V1 149, V2 139
    (19, "b16", 0, 1, 1, 256, 125, 125, 1, 4),    # V1 64, V2 73
    (27, "b16", 6, 1, 0, 384, 103, 101, 2, 3),    # V2 131, one node per thread 139
    (27, "b16", 0, 1, 0, 384, 103, 101, 0, 0),    # V2 slower by a quarter
    (27, "b16", 6, 1, 0, 448, 19, 18, 1, 7),      # 11.1, one node per thread 11.8
    (27, "b16", 6, 1, 0, 448, 95, 94, 0, 0),
    (19, "f64", 0, 1, 1, 320, 15, 12, 1, 5),      # 7.9, 8.6
    (19, "f64", 0, 1, 1, 320, 23, 20, 1, 5),      # 12.5, 13.3
    (19, "f64", 0, 1, 1, 320, 113, 111, 0, 0),    # 283, 256
    (19, "f64", 0, 1, 0, 448, 15, 15, 1, 7),      # 9.3, 10.3
    (19, "f64", 0, 1, 0, 448, 9, 7, 0, 0),        # 7.2, 6.5
    (19, "f64", 0, 1, 0, 448, 31, 29, 0, 0),      # 27.4, 22.1
    (27, "f64", 0, 2, 1, 256, 15, 16, 1, 4),      # 13.6, 15.7
    (27, "f64", 0, 2, 1, 256, 25, 23, 0, 0),      # 34.7, 29.6
    (27, "f64", 0, 2, 1, 64, 31, 30, 1, 1),       # 11.4, 13.9
    (19, "f32", 0, 2, 1, 320, 23, 20, 1, 5),      # 8.9, 10.5
    (19, "f32", 0, 2, 1, 320, 15, 12, 0, 0),      # 7.6, 6.9
    (19, "f32", 0, 2, 1, 320, 113, 111, 0, 0),    # 165, 156
    (19, "f64", 0, 0, 0, 512, 11, 11, 1, 8),      # V1 7.9, V2 8.2
    (19, "f64", 0, 0, 0, 512, 128, 128, 2, 4),
]


@pytest.mark.parametrize("case", CHOICES, ids=lambda c: "-".join(str(v) for v in c[:8]))
def test_kernel_is_the_faster_measured_one(case):
    q, V, W = case[0], case[8], case[9]
    assert ask(["vec " + " ".join(str(v) for v in case[1:8])], q)[0] == [V, W, 0]
