"""Launch shapes of the one-node-per-thread kernels, from the library's own rule on the host: every
node has exactly one thread at every row length, and the layout is the one that was measured to be
faster at shapes on both sides of the rule's lines."""
import pytest

from launch_plan import ask

SR = 2 | 4  # FP32 rest and stochastic rounding


def test_every_node_has_one_thread():
    lines = [f"rows {form} {flags} {u} {root} {nx} {ny} {nz}"
             for form, flags, u, root in [("f64", 0, 2, 0), ("f32", 0, 1, 0), ("b16", SR, 0, 0), ("f32", 0, 0, 1)]
             for nx in list(range(1, 132)) + [192, 255, 256, 257, 511, 512, 513, 1025]
             for ny, nz in [(1, 1), (2, 300), (17, 16), (61, 61), (300, 600)]]
    for line, (rows, pitch, threads, gx, gy, gz, covered) in zip(lines, ask(lines)):
        nx, ny, nz = (int(v) for v in line.split()[-3:])
        assert covered == 1 and gz == nz, line
        assert threads % 64 == 0 and threads <= 512 and gx * threads >= nx, line
        assert gy <= (ny + rows - 1) // rows, line


# (form, flags, velocity mode, nx, ny, nz) -> rows, threads per row. Times in us per step of the two
# layouts, FP32 and FP64 with a constant velocity unless the velocity mode says otherwise
PADDED = [("f32", 0, 1, 90, 200, 150, 2, 128),     # 89.3 padded, 91.4 alone
          ("f32", 0, 1, 90, 300, 300, 2, 128),     # 319, 322
          ("f64", 0, 1, 90, 300, 300, 2, 128),     # 563, 576
          ("f32", 0, 1, 33, 349, 347, 4, 64),      # 134, 176 packed
          ("f32", 0, 1, 20, 447, 447, 8, 32),      # 126, 158
          ("b16", 0, 0, 50, 283, 283, 4, 64),      # 67, 81
          ("f32", 0, 1, 110, 37, 37, 2, 128),      # 8.3, 9.4 alone
          ("f32", 0, 1, 40, 61, 61, 4, 64)]        # 6.3, 7.8 packed
PACKED = [("f64", 0, 1, 32, 32, 32, 4, 32),        # 6.6 padded, 5.4 in 256 small blocks
          ("f64", 0, 2, 90, 200, 150, 2, 128),     # FP64 with a velocity field: as padded
          ("f64", 0, 2, 70, 239, 239, 3, 70),      # 1.22 times as fast packed
          ("b16", SR, 1, 70, 239, 239, 3, 70),     # 1.28
          ("b16", 0, 1, 70, 239, 239, 3, 70),      # 79 us, padded 99 (porous)
          ("b16", 0, 1, 18, 119, 117, 7, 18),      # 7.9 in blocks of two wavefronts, padded 9.4
          ("f32", 0, 1, 70, 120, 120, 3, 70),      # 1.06
          ("b16", SR, 1, 110, 191, 190, 1, 110)]   # 1.07 alone


@pytest.mark.parametrize("form,flags,u,nx,ny,nz,rows,pitch", PADDED + PACKED)
def test_layout_is_the_faster_measured_one(form, flags, u, nx, ny, nz, rows, pitch):
    got = ask([f"rows {form} {flags} {u} 0 {nx} {ny} {nz}"])[0]
    assert got[:2] == [rows, pitch]


def test_gpu_test_lattices_take_their_layouts():
    import test_gpu_row_layouts as t
    for prec, opts, velocity, nx, ny, nz, parts, rows, pitch in t.CASES:
        form = prec if prec in ("f64", "f32") else "b16"
        head = f"rows {form} {2 if opts else 0} {2 if velocity == 'field' else 1} 0 {nx} {ny}"
        whole, part = ask([f"{head} {nz}", f"{head} {nz // parts}"])
        assert whole[:2] == [rows, pitch] and part[:2] != whole[:2], head


@pytest.mark.parametrize("form,flags", [("f64", 0), ("f32", 0), ("b16", 0), ("b16", SR)])
def test_long_planes_stay_within_a_grid(form, flags):
    """Rows up to 128 nodes in a plane of 131 070 rows (65 535 blocks of two), which padded rows
    reach: no layout has more blocks in y than a grid takes."""
    lines = [f"rows {form} {flags} 1 0 {nx} 131070 1" for nx in (1, 16, 17, 32, 33, 64, 65, 85, 90, 97, 110, 128)]
    for line, (rows, pitch, threads, gx, gy, gz, covered) in zip(lines, ask(lines)):
        assert gy <= 65535 and covered == 1, line
