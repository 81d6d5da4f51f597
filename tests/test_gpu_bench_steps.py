"""The benchmark asks the lattice's buffers how many steps a launch takes, not a file: two where the
library pairs steps, one where a flag names the single-step kernel, at odd and even parities of the
steps taken before."""
import os
import sys

import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402
from paper_2605_01774_amd import inputs as I, lattice  # noqa: E402
from gpuhelp import banner  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("before", [0, 1])
@pytest.mark.parametrize("prec,kw,want", [("f32", {}, 2), ("f64", {}, 2), ("f32", dict(scalar_kernel=True), 1),
                                          ("bf16", {}, 1), ("bf16", dict(rest_fp32=True, stochastic_rounding=True), 1)])
def test_steps_per_launch(prec, kw, want, before):
    banner(f"bench: steps per launch {prec} {kw} after {before}")
    prob = I.fourier_decay(n=128, steps=1, precision=prec)
    lat = lattice.from_problem(prob, precision=prec, device="cuda:0", **kw)
    lat.step(before)
    init = lat.save_state()
    assert bench.steps_per_launch(lat, init) == want
    lat.load_state(*init)
    torch.cuda.synchronize()
