"""Two steps in one launch against single steps, over the coefficients and tiles that the two-step
kernel accepts: tensor fields and source fields, together and alone, on tiles of whole rows and on
tiles with halo columns, between walls and periodic; and a source amplitude that changes between two
paired runs. Bitwise equal states, counters and records.

Every case checks that its run took two steps per launch: the buffer that the state is not in then
holds the state two steps back, where single steps leave the state one step back."""
import numpy as np
import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu

# (nx, ny, nz) -> tensor, source, boundary. Whole rows and tiles with halo columns (176 and more in
# FP64, 353 and more in FP32), sizes that no tile divides
CASES = [("f64", (128, 121, 128), "field", "field"), ("f64", (160, 151, 160), "field", "field"),
         ("f64", (240, 163, 160), "field", "none"), ("f64", (256, 101, 240), "field", "field"),
         ("f64", (176, 131, 160), "uniform", "field"), ("f64", (353, 80, 83), "table", "field"),
         ("f64", (64, 211, 203), "uniform", "none"), ("f64", (231, 160, 160), "field", "uniform"),
         ("f32", (128, 121, 128), "field", "field"), ("f32", (160, 151, 160), "field", "field"),
         ("f32", (200, 151, 131), "uniform", "field"), ("f32", (353, 151, 140), "table", "field"),
         ("f32", (320, 157, 160), "field", "field"), ("f32", (96, 96, 99), "table", "none"),
         ("f32", (144, 99, 131), "uniform", "uniform")]
T_MODE = {"uniform": 0, "field": 1, "table": 2}
R_MODE = {"none": 0, "uniform": 1, "field": 2}


def _lattice(shape, prec, tensor, source, bc, scalar, background=1.0):
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(3)

    def rnd(*s):
        return torch.rand(*s, generator=gen, dtype=torch.float64, device="cuda:0")

    lat = lattice.Lattice(nx, ny, nz, precision=prec, bc_x=bc, phi_ref=background, eps=0.0 if background else 1e-6,
                          device="cuda:0", scalar_kernel=scalar)
    table = np.array([[1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3], [1e-1, 0, 0, 1e-2, 0, 1e-4], [2e-3, 0, 1e-4, 2e-3, 0, 1e-2]])
    if tensor == "uniform":
        lat.set_diffusion(table[0])
    elif tensor == "table":
        lat.set_diffusion_phases(table, (rnd(nz, ny, nx) * 3).to(torch.uint8))
    else:
        lat.set_diffusion(torch.as_tensor(table[0], device="cuda:0")[:, None, None, None] * (0.5 + rnd(1, nz, ny, nx)))
    lat.set_velocity([0.0, 0.0, 0.0])
    if source == "field":
        lat.set_source(1e-3 * (rnd(nz, ny, nx) - 0.5))
    elif source == "uniform":
        lat.set_source(2e-4)
    if bc == "dirichlet":
        lat.set_dirichlet(1.3, 0.8)
    lat.init_equilibrium(background + 0.2 * rnd(nz, ny, nx) if background else (rnd(nz, ny, nx) > 0.9).double())
    return lat


def _took_pairs(lat, two_back):
    """Whether the lattice's last run of four steps, from a fresh start, took two per launch; two_back:
    the raw state two steps before its end."""
    cur = lat.save_state()[0]
    at_a = torch.equal(lat.buf_a, cur)
    assert at_a or torch.equal(lat.buf_b, cur)
    return torch.equal(lat.buf_b if at_a else lat.buf_a, two_back)


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("prec,shape,tensor,source", CASES)
def test_two_steps_per_launch_bitwise(prec, shape, tensor, source, bc):
    banner(f"two steps per launch {prec} {shape} {tensor} {source} {bc}")
    ref = _lattice(shape, prec, tensor, source, bc, True)
    lat = _lattice(shape, prec, tensor, source, bc, False)
    ref.step(2)
    two_back = ref.save_state()[0]
    ref.step(2)
    lat.step(4)
    assert _took_pairs(lat, two_back)
    del two_back
    # the amplitude of a source changes while its second half-step is pending
    for scale, n in ((0.25, 5), (1.5, 8)):
        for x in (ref, lat):
            if source != "none":
                x.set_source_scale(scale)
            x.step(n)
        assert torch.equal(lat.save_state()[0], ref.save_state()[0]), n
        assert lat.counters() == ref.counters()


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("prec,shape,tensor", [("f64", (240, 163, 160), "field"), ("f64", (64, 211, 203), "uniform"),
                                               ("f32", (320, 157, 160), "field"), ("f32", (96, 96, 99), "table")])
def test_records_and_fallback(prec, shape, tensor, bc):
    """A zero background with eps > 0: the fallback and the guard act; records of a run of seven steps,
    four of them in pairs."""
    banner(f"two steps per launch, records {prec} {shape} {tensor} {bc}")
    out = []
    for scalar in (True, False):
        lat = _lattice(shape, prec, tensor, "none", bc, scalar, background=0.0)
        lam = torch.empty(7 * lat.n, dtype=lat.real, device="cuda:0")
        br = torch.empty(7 * lat.n, dtype=torch.uint8, device="cuda:0")
        lat.step_record(7, lam, br)
        out.append((lam, br, lat.save_state()[0], lat.counters()))
        del lat
    for a, b in zip(out[0][:3], out[1][:3]):
        assert torch.equal(a, b)
    assert out[0][3] == out[1][3] and out[0][3]["fallback_nodes"] > 0
