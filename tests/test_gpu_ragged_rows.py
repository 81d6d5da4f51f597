"""Row-vector kernel on rows that are no multiple of a wavefront, against the one-node-per-thread
kernel (scalar_kernel=True, which other tests compare with the oracle): bitwise equal states,
counters and records, at the row lengths where its last wavefront is nearly empty, full or one
node over, where a row needs one wavefront, several and the most it takes, and beyond."""
import numpy as np
import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu

FORMS = {"f64": ("f64", {}), "f32": ("f32", {}), "bf16": ("bf16", {}), "fp16": ("fp16", {}),
         "bf16r": ("bf16", dict(rest_fp32=True, stochastic_rounding=True)),
         "fp16r": ("fp16", dict(rest_fp32=True, stochastic_rounding=True))}


def _run(nx, form, kind, bc, q, scalar):
    ny, nz = 5, 4
    prec, opts = FORMS[form]
    gen = torch.Generator(device="cuda:0").manual_seed(nx)

    def rnd(*s):
        return torch.rand(*s, generator=gen, dtype=torch.float64, device="cuda:0")

    background = 0.0 if kind == "uniform" else 1.0
    lat = lattice.Lattice(nx, ny, nz, precision=prec, bc_x=bc, phi_ref=background, eps=1e-6, device="cuda:0", q=q,
                          scalar_kernel=scalar, **opts)
    d6 = np.array([1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3])
    if kind == "uniform":
        lat.set_diffusion(d6)
        lat.set_velocity([0.04, -0.02, 0.03])
        phi0 = (rnd(nz, ny, nx) > 0.8).double()
    elif kind == "table":
        lat.set_diffusion_phases(np.stack([d6, 3 * d6]), (rnd(nz, ny, nx) * 2).to(torch.uint8))
        lat.set_velocity([0.0, 0.0, 0.0])
        phi0 = 1.0 + 0.2 * rnd(nz, ny, nx)
    else:
        lat.set_diffusion(torch.as_tensor(d6, device="cuda:0")[:, None, None, None] * (0.5 + rnd(1, nz, ny, nx)))
        lat.set_velocity(0.08 * (rnd(3, nz, ny, nx) - 0.5))
        lat.set_source(1e-3 * (rnd(nz, ny, nx) - 0.5))
        phi0 = 1.0 + 0.2 * rnd(nz, ny, nx)
    if bc == "dirichlet":
        lat.set_dirichlet(1.3, 0.8)
    lat.init_equilibrium(phi0)
    lat.step(3)
    out = [lat.save_state()[0].cpu(), lat.counters()]
    if not opts:
        lam = torch.empty(lat.n, dtype=lat.real, device="cuda:0")
        br = torch.empty(lat.n, dtype=torch.uint8, device="cuda:0")
        lat.step_record(1, lam, br)
        out += [lam.cpu(), br.cpu()]
    return out


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("kind", ["uniform", "table", "field"])
@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("q", [19, 27])
def test_ragged_rows_bitwise(q, form, kind, bc):
    banner(f"ragged rows q{q} {form} {kind} {bc}")
    for nx in (1, 2, 3, 10, 62, 63, 65, 66, 126, 129, 130, 200, 254, 258, 322, 449, 510, 514, 1022, 1026):
        ref = _run(nx, form, kind, bc, q, True)
        got = _run(nx, form, kind, bc, q, False)
        assert torch.equal(got[0], ref[0]), nx
        assert got[1] == ref[1], nx
        for a, b in zip(got[2:], ref[2:]):
            assert torch.equal(a, b), nx


@pytest.mark.parametrize("prec,nx,ny,nz", [("f64", 105, 95, 92), ("f64", 81, 105, 108), ("f64", 33, 161, 164),
                                           ("f32", 81, 145, 148), ("f32", 105, 121, 140)])
def test_rows_of_large_lattices(prec, nx, ny, nz):
    """Rows are laid out over blocks by another rule beyond 128 MB of state: a lattice over that
    size of two equal halves in z against one of half the size, bitwise."""
    banner(f"rows of a large lattice {nx}x{ny}x{nz} {prec}")
    per = 19 * (8 if prec == "f64" else 4)
    assert nx * ny * nz * per > 128e6 > nx * ny * (nz // 2) * per
    gen = torch.Generator(device="cuda:0").manual_seed(nx)
    half = 1.0 + 0.2 * torch.rand(nz // 2, ny, nx, generator=gen, dtype=torch.float64, device="cuda:0")
    out = []
    for phi0 in (half, torch.cat([half, half])):
        lat = lattice.Lattice(nx, ny, phi0.shape[0], precision=prec, phi_ref=1.0, device="cuda:0")
        lat.set_diffusion([1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3])
        lat.set_velocity([0.04, -0.02, 0.03])
        lat.init_equilibrium(phi0)
        lat.step(3)
        out.append(lat.populations())
    assert torch.equal(out[1], torch.cat([out[0], out[0]], dim=1))
