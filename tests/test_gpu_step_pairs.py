"""Two steps in one launch against single steps: bitwise equal states, counters and records.

The reference is the one-node-per-thread kernel (scalar_kernel=True), which the other tests
compare with the oracle. The lattices are of sizes at which elbm_step takes two steps per
launch: tiles across whole rows and tiles with halo columns, remainders in x, y and z, a last
sweep shorter than the others, the smallest sizes of the range, odd step counts (the last
step single), and both kinds of node that the second step reads from its own column (walls)
or across the periodic seam."""
import numpy as np
import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu


def _lattice(shape, prec, tensor, bc, source, scalar, seed=11, background=1.0, eps=0.0):
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(seed)

    def rnd(*s):
        return torch.rand(*s, generator=gen, dtype=torch.float64, device="cuda:0")

    lat = lattice.Lattice(nx, ny, nz, precision=prec, bc_x=bc, phi_ref=background, eps=eps, device="cuda:0",
                          scalar_kernel=scalar)
    table = np.array([[1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3], [1e-1, 0, 0, 1e-2, 0, 1e-4],
                      [2e-3, 0, 1e-4, 2e-3, 0, 1e-2]])
    if tensor == "uniform":
        lat.set_diffusion(table[0])
    elif tensor == "table":
        lat.set_diffusion_phases(table, (rnd(nz, ny, nx) * 3).to(torch.uint8))
    else:
        d6 = torch.as_tensor(table[0], device="cuda:0")[:, None, None, None] * (0.5 + rnd(1, nz, ny, nx))
        lat.set_diffusion(d6)
    lat.set_velocity([0.0, 0.0, 0.0])
    if source == "field":
        lat.set_source(1e-3 * (rnd(nz, ny, nx) - 0.5))
    elif source == "uniform":
        lat.set_source(2e-4)
    if bc == "dirichlet":
        lat.set_dirichlet(1.3, 0.8)
    phi0 = background + 0.2 * rnd(nz, ny, nx) if background else (rnd(nz, ny, nx) > 0.9).double()
    lat.init_equilibrium(phi0, 0.05 * (rnd(3, nz, ny, nx) - 0.5) * phi0)
    return lat


def _state(lat):
    raw, step, pending = lat.save_state()
    return raw.cpu(), step, pending, lat.counters()


def _same(a, b):
    assert torch.equal(a[0], b[0])
    assert a[1:] == b[1:]


# (nx, ny, nz): whole-row tiles (96 to 200 in FP32, 96 and 100 in FP64), tiles with halo
# columns (353 in FP32, 176 and 240 in FP64), sizes that no tile divides
SHAPES = {"f32": [(96, 96, 96), (99, 97, 131), (128, 128, 121), (200, 151, 67), (353, 128, 128)],
          "f64": [(96, 97, 96), (100, 90, 113), (176, 120, 83), (240, 176, 96)]}


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("tensor,source", [("uniform", "none"), ("field", "field"), ("table", "uniform")])
@pytest.mark.parametrize("prec,shape", [(p, s) for p in SHAPES for s in SHAPES[p]])
def test_two_steps_per_launch_bitwise(prec, shape, tensor, source, bc):
    banner(f"two steps per launch {prec} {shape} {tensor} {source} {bc}")
    ref = _lattice(shape, prec, tensor, bc, source, True)
    lat = _lattice(shape, prec, tensor, bc, source, False)
    for n in (2, 5):
        ref.step(n)
        lat.step(n)
        _same(_state(lat), _state(ref))


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("prec,shape", [("f32", (200, 151, 67)), ("f64", (96, 97, 96))])
def test_two_steps_per_launch_fallback_and_records(prec, shape, bc):
    """A zero background with eps > 0: the positivity fallback and the phi <= 0 guard act, and
    their counts, lambda and branches agree step by step."""
    banner(f"two steps per launch, records {prec} {shape} {bc}")
    out = []
    for scalar in (True, False):
        lat = _lattice(shape, prec, "field", bc, "none", scalar, background=0.0, eps=1e-6)
        lam = torch.empty(4 * lat.n, dtype=lat.real, device="cuda:0")
        br = torch.empty(4 * lat.n, dtype=torch.uint8, device="cuda:0")
        lat.step_record(4, lam, br)
        out.append((lam.cpu(), br.cpu(), _state(lat)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    _same(out[1][2], out[0][2])
    assert out[0][2][3]["fallback_nodes"] > 0
