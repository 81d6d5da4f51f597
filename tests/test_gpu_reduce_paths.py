"""Global sums and the smallest population where the reduction changes from one launch to two (512 blocks
of 256 nodes), on both sides of the line and at most blocks: equal to the two-launch sums of
reduce_noalloc bitwise, to exact sums of the readout within rounding, to the smallest population read
out, and the same on repeated calls between which the state and the other reduction move on."""
import math

import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32", "fp16"])
@pytest.mark.parametrize("shape", [(64, 64, 32), (131073, 1, 1), (71, 47, 40), (257, 64, 33)])  # 512, 513, 522, 2121 -> 2048
def test_reductions_on_both_sides_of_one_launch(shape, prec):
    banner(f"reduction paths {shape} {prec}")
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(8)
    lat = lattice.Lattice(nx, ny, nz, precision=prec, phi_ref=1.5, device="cuda:0")
    lat.set_diffusion([2e-2, 1e-3, 0, 1e-2, 0, 5e-3])
    lat.set_velocity([0.02, -0.01, 0.03])
    lat.set_source(1e-3)
    lat.init_equilibrium(1.0 + torch.rand(nz, ny, nx, generator=gen, dtype=torch.float64, device="cuda:0"))
    dev = torch.empty(4, dtype=torch.float64, device="cuda:0")
    for _ in range(3):
        lat.step(1)
        got = lat.reduce()
        lat.reduce_noalloc(dev)
        assert torch.equal(dev.cpu(), torch.from_numpy(got))
        assert lat.min_population() == float(lat.populations().min())
        assert (lat.reduce() == got).all()
    phi = lat.moments()[0].reshape(-1).tolist()
    # compensated per thread, then at most 6 + 3 + 8 + 6 + 3 roundings of partial sums
    assert abs(got[0] - math.fsum(phi)) <= 32 * 2.0 ** -53 * math.fsum(abs(v) for v in phi)
