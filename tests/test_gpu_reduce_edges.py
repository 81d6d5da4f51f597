"""Global sums and the smallest population at the edges of the reduction's blocks: one node,
one more and one less than a wavefront, a block and the most blocks of the first pass (2048
of 256 nodes), against exact sums of the readouts; and repeated calls, between which the
blocks' ticket runs on."""
import math

import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 1, 1), (65, 1, 1), (255, 1, 1), (257, 1, 1), (128, 64, 64),
                                   (131, 64, 63)])
def test_reduce_at_block_edges(shape, prec):
    banner(f"reduction edges {shape} {prec}")
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    phi0 = 1.0 + torch.rand(nz, ny, nx, generator=gen, dtype=torch.float64, device="cuda:0")
    j0 = 0.01 * (torch.rand(3, nz, ny, nx, generator=gen, dtype=torch.float64, device="cuda:0") - 0.5)
    lat = lattice.Lattice(nx, ny, nz, precision=prec, phi_ref=1.5, device="cuda:0")
    lat.set_diffusion([2e-2, 1e-3, 0, 1e-2, 0, 5e-3])
    lat.set_velocity([0.02, -0.01, 0.03])
    lat.set_source(1e-3)
    lat.init_equilibrium(phi0, j0)
    lat.step(1)
    phi, q = lat.moments()
    sums = [math.fsum(t.reshape(-1).tolist()) for t in (phi, q[0], q[1], q[2])]
    # compensated per thread, then at most 6 + 3 + 8 + 6 + 3 roundings of partial sums; the
    # readout rounds phi_ref + dphi once per node, which the reduction does not
    scale = [math.fsum(t.abs().reshape(-1).tolist()) for t in (phi, q[0], q[1], q[2])]
    for _ in range(3):
        got = lat.reduce()
        for m in range(4):
            assert abs(got[m] - sums[m]) <= 32 * 2.0 ** -53 * scale[m] + 1e-300
        dev = torch.empty(4, dtype=torch.float64, device="cuda:0")
        lat.reduce_noalloc(dev)
        assert torch.equal(dev.cpu(), torch.from_numpy(got))
        assert lat.min_population() == float(lat.populations().min())


def test_reduce_beside_noalloc_on_another_stream():
    """The sums that the host waits for and those of reduce_noalloc count their blocks apart, so
    one may run while the other is in flight on another stream."""
    banner("reduction beside a reduction on another stream")
    lat = lattice.Lattice(128, 128, 64, precision="f32", phi_ref=1.0, device="cuda:0")
    lat.set_diffusion([2e-2, 1e-3, 0, 1e-2, 0, 5e-3])
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    lat.init_equilibrium(1.0 + torch.rand(64, 128, 128, generator=gen, dtype=torch.float64, device="cuda:0"))
    want = lat.reduce()
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    dev = torch.zeros(20, 4, dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    for k in range(20):
        lat.set_stream(one)
        lat.reduce_noalloc(dev[k])
        lat.set_stream(two)
        assert (lat.reduce() == want).all()
    torch.cuda.synchronize()
    assert (dev.cpu().numpy() == want).all()
