"""Layouts of the one-node-per-thread kernels and of the adjoint: a lattice of equal parts in z, large
enough for padded, packed and single rows in 256-thread blocks, against one part alone, whose few rows
take another layout: bitwise equal states, and gradients. Which layouts they are is checked on the host
(test_row_layouts_cpu.py)."""
import numpy as np
import pytest
import torch

from paper_2605_01774_amd import lattice
from paper_2605_01774_amd.autograd import AdjointRun
from gpuhelp import banner

pytestmark = pytest.mark.gpu

ROUNDING = dict(rest_fp32=True)  # stochastic rounding draws by node, so it differs between the parts

# (precision, options, velocity, nx, ny, nz, parts) -> rows of a block, threads of a row
CASES = [("f64", {}, "uniform", 33, 67, 68, 4, 7, 33), ("f32", {}, "uniform", 85, 60, 60, 4, 3, 85),
         ("f32", {}, "uniform", 55, 60, 64, 16, 4, 64), ("f32", {}, "uniform", 110, 61, 64, 32, 2, 128),
         ("bf16", {}, "field", 40, 126, 128, 16, 6, 40), ("bf16", ROUNDING, "uniform", 20, 121, 120, 4, 12, 20),
         ("fp16", ROUNDING, "uniform", 110, 131, 128, 16, 1, 110), ("fp16", ROUNDING, "uniform", 75, 131, 128, 64, 3, 75), ("bf16", {}, "uniform", 18, 119, 120, 60, 10, 18),
         ("f64", {}, "field", 70, 120, 128, 32, 3, 70), ("f64", {}, "uniform", 32, 32, 32, 2, 4, 32)]


def _parts(shape, parts, seed):
    """Arrays of one part and of the whole lattice."""
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(seed)

    def rnd(c):
        one = torch.rand(c, nz // parts, ny, nx, generator=gen, dtype=torch.float64, device="cuda:0")
        return one, one.repeat(1, parts, 1, 1)

    return rnd


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{'x'.join(map(str, c[3:6]))}-{c[2]}")
def test_parts_equal_the_whole(case):
    prec, opts, velocity, nx, ny, nz, parts, rows, pitch = case
    banner(f"row layouts {prec} {nx}x{ny}x{nz} {velocity}")
    rnd = _parts((nx, ny, nz), parts, nx)
    phi, u = rnd(1), rnd(3)
    out = []
    for k in (0, 1):
        lat = lattice.Lattice(nx, ny, nz if k else nz // parts, precision=prec, phi_ref=1.0, device="cuda:0",
                              scalar_kernel=True, **opts)
        lat.set_diffusion([1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3])
        lat.set_velocity(0.08 * (u[k] - 0.5) if velocity == "field" else [0.04, -0.02, 0.03])
        lat.init_equilibrium(1.0 + 0.2 * phi[k][0])
        lat.step(3)
        out.append(lat.populations())
    assert torch.equal(out[1], out[0].repeat(1, parts, 1, 1))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,nz", [(33, 67, 68), (85, 61, 60), (110, 61, 64), (20, 81, 80)])
def test_gradient_of_parts_equals_the_whole(nx, ny, nz, prec):
    banner(f"row layouts, adjoint {prec} {nx}x{ny}x{nz}")
    rnd = _parts((nx, ny, nz), 4, nx + 1)
    phi, d, g = rnd(1), rnd(1), rnd(1)
    d6 = torch.as_tensor(np.array([1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3]), device="cuda:0")[:, None, None, None]
    out = []
    for k in (0, 1):
        lat = lattice.Lattice(nx, ny, nz if k else nz // 4, precision=prec, phi_ref=1.0, device="cuda:0")
        lat.set_diffusion(d6 * (0.5 + d[k]))
        lat.set_velocity([0.03, 0.0, -0.02])
        lat.init_equilibrium(1.0 + 0.2 * phi[k][0])
        run = AdjointRun(lat, 5, 2)
        run.forward()
        t = run.backward(g[k][0])
        out.append((t.reshape(-1, ny * nx, 6), run.dphi0))
    assert torch.equal(out[1][0], out[0][0].repeat(4, 1, 1))
    assert torch.equal(out[1][1], out[0][1].repeat(4, 1, 1))
