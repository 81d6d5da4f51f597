"""elbm_step captured in a HIP graph and replayed: every replay advances the state by the captured
steps, bitwise as direct steps do, whether the library takes one step per launch or two. A call of an
even number of steps leaves the state in the buffer it started from, which is what makes it
replayable; so the buffer that holds the state after any call follows the parity of its steps."""
import pytest
import torch

from paper_2605_01774_amd import lattice
from gpuhelp import banner

pytestmark = pytest.mark.gpu


def _lattice(shape, prec, scalar=False, **opts):
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda:0").manual_seed(17)
    lat = lattice.Lattice(nx, ny, nz, precision=prec, phi_ref=1.0, device="cuda:0", scalar_kernel=scalar, **opts)
    lat.set_diffusion([1e-2, 2e-3, -1e-3, 8e-3, 1e-3, 5e-3])
    lat.set_velocity([0.0, 0.0, 0.0])
    lat.set_source(2e-4)
    lat.init_equilibrium(1.0 + 0.2 * torch.rand(nz, ny, nx, generator=gen, dtype=torch.float64, device="cuda:0"))
    return lat


# two steps per launch (128^3), single steps of the one-node-per-thread (37 x 24 x 20, 16-bit) and
# row-vector kernels (64 x 16 x 16)
CASES = [("f32", (128, 128, 128)), ("f64", (128, 128, 128)), ("f32", (37, 24, 20)), ("f64", (64, 16, 16)),
         ("bf16", (64, 16, 16))]


@pytest.mark.parametrize("n", [2, 4, 6, 10])
@pytest.mark.parametrize("prec,shape", CASES)
def test_replays_advance_the_state(prec, shape, n):
    banner(f"captured step({n}) {prec} {shape}")
    lat, ref = _lattice(shape, prec), _lattice(shape, prec, scalar=True)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    lat.set_stream(stream)
    lat.step(n)
    ref.step(n)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        lat.step(n)
    for replay in range(3):
        graph.replay()
        torch.cuda.synchronize()
        ref.step(n)
        got, want = lat.save_state()[0], ref.save_state()[0]
        torch.cuda.synchronize()
        assert torch.equal(got, want), replay


@pytest.mark.parametrize("prec,shape", CASES[:3])
def test_state_lies_in_the_buffer_of_the_steps_parity(prec, shape):
    banner(f"buffer after a run {prec} {shape}")
    lat = _lattice(shape, prec)
    total = 0
    for n in (1, 2, 3, 4, 5, 6, 7, 8):
        lat.step(n)
        total += n
        state = lat.save_state()[0]
        assert torch.equal((lat.buf_a, lat.buf_b)[total % 2], state), n
