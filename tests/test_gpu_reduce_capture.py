"""elbm_reduce_noalloc uses the caller's buffers and the library's static array only: captured calls
of two lattices are replayed after both handles are gone, with steps of a third lattice (whose scratch
may lie where theirs lay) and its own reductions between the replays, and give the sums of the
buffers as they are then. The third lattice's counters show that nothing wrote into its scratch."""
import numpy as np
import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu


def _lattice(shape, prec, seed):
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    lat = lattice.Lattice(nx, ny, nz, precision=prec, phi_ref=1.0, device="cuda:0")
    lat.set_diffusion([2e-2, 1e-3, 0, 1e-2, 0, 5e-3])
    lat.set_velocity([0.02, -0.01, 0.03])
    lat.init_equilibrium(1.0 + torch.rand(nz, ny, nx, generator=gen, dtype=torch.float64, device="cuda:0"))
    lat.step(2)
    return lat


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_captured_reduction_outlives_its_handle(prec):
    banner(f"captured reductions after their handles {prec}")
    stream = torch.cuda.Stream()
    graphs, outs, wants, lats = [], [], [], []
    for k, shape in enumerate([(40, 24, 20), (65, 13, 7)]):  # 75 and 24 block partials
        lat = _lattice(shape, prec, k)
        wants.append(lat.reduce())
        out = torch.zeros(4, dtype=torch.float64, device="cuda:0")
        torch.cuda.synchronize()
        lat.set_stream(stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            lat.reduce_noalloc(out)
        graphs.append(graph)
        outs.append(out)
        lats.append(lat)
    for lat in lats:  # the handles go, the buffers stay with the Python objects
        lat.close()
    other = _lattice((40, 24, 20), prec, 5)
    other.reset_counters()
    for replay in range(3):
        for graph, out, want in zip(graphs, outs, wants):
            out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want), replay
        other.step(1)
        dev = torch.empty(4, dtype=torch.float64, device="cuda:0")
        other.reduce_noalloc(dev)
        assert np.array_equal(dev.cpu().numpy(), other.reduce())
    assert other.counters() == dict(fallback_nodes=0, flagged_nodes=0, nonfinite=0, guard_nodes=0)
