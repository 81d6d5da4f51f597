"""The row-vector kernel's form for ragged rows (16-bit storage with FP32 rest or stochastic rounding,
u = 0, on lattices that fill the chip) against the one-node-per-thread kernel: bitwise equal states,
counters, lambda and branch records. Rows of one to eight wavefronts, the last of them full, nearly
full, or with the fewest lanes the form takes; row counts that its blocks of four or two rows do not
divide. That the form is the one that runs at these shapes is checked on the host
(test_ragged_rule_cpu.py)."""
import numpy as np
import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu

# (nx, ny, nz): 1, 1, 2, 2, 2, 3, 4, 4 wavefronts in both velocity sets; 6 and 8 in D3Q19
SHAPES = [(100, 79, 79), (126, 77, 81), (194, 55, 57), (200, 55, 57), (254, 55, 57), (290, 45, 47), (386, 39, 41),
          (510, 39, 41)]
LONG = [(642, 59, 59), (1022, 51, 51)]
STORAGE = {"both": dict(rest_fp32=True, stochastic_rounding=True), "rest": dict(rest_fp32=True),
           "rounding": dict(stochastic_rounding=True)}
KINDS = {"uniform": dict(), "uniform, source field": dict(source="field"), "two materials, source": dict(phases=2, source="uniform"),
         "five materials, source field": dict(phases=5, source="field"), "fallback": dict(background=0.0)}


def _run(shape, prec, storage, q, bc, scalar, phases=0, source=None, background=1.0):
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(nx)

    def rnd(*s):
        return torch.rand(*s, generator=gen, dtype=torch.float64, device="cuda:0")

    lat = lattice.Lattice(nx, ny, nz, precision=prec, bc_x=bc, phi_ref=background, eps=0.0 if background else 1e-6,
                          device="cuda:0", q=q, scalar_kernel=scalar, **STORAGE[storage])
    d6 = np.array([1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3])
    if phases:
        lat.set_diffusion_phases(np.stack([d6 * (m + 1) for m in range(phases)]), (rnd(nz, ny, nx) * phases).to(torch.uint8))
    else:
        lat.set_diffusion(d6)
    lat.set_velocity([0.0, 0.0, 0.0])
    if source == "field":
        lat.set_source(1e-3 * (rnd(nz, ny, nx) - 0.5))
    elif source:
        lat.set_source(2e-4)
    if bc == "dirichlet":
        lat.set_dirichlet(1.3, 0.8)
    lat.init_equilibrium(background + 0.2 * rnd(nz, ny, nx) if background else (rnd(nz, ny, nx) > 0.9).double())
    lat.step(2)
    lam = torch.empty(2 * lat.n, dtype=lat.real, device="cuda:0")
    br = torch.empty(2 * lat.n, dtype=torch.uint8, device="cuda:0")
    lat.step_record(2, lam, br)
    return lat.save_state()[0], lam, br, lat.counters()


def _check(shape, prec, storage, q, bc, kind):
    banner(f"ragged form q{q} {shape} {prec} {storage} {kind} {bc}")
    got = _run(shape, prec, storage, q, bc, False, **KINDS[kind])
    ref = _run(shape, prec, storage, q, bc, True, **KINDS[kind])
    for a, b in zip(got[:3], ref[:3]):
        assert torch.equal(a, b)
    assert got[3] == ref[3]
    if kind == "fallback":
        assert got[3]["fallback_nodes"] > 0


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("q", [19, 27])
def test_ragged_form_bitwise(q, kind, bc):
    for k, shape in enumerate(SHAPES + (LONG if q == 19 else [])):
        _check(shape, ("bf16", "fp16")[k % 2], sorted(STORAGE)[k % 3], q, bc, kind)


@pytest.mark.parametrize("storage", sorted(STORAGE))
@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_every_storage_option(prec, storage):
    for bc, kind in (("periodic", "uniform, source field"), ("dirichlet", "five materials, source field")):
        _check((194, 55, 57), prec, storage, 19, bc, kind)
