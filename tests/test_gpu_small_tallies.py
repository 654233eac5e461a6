"""Tallies of small launches (workgroups of 256 particles, tables of 512 cells) against those of the
same histories in one large launch or in many: edges of a workgroup and of the rule between the
two (128 particles to a compute unit).  The order of FP64 additions is all that may differ: 1e-12
of the cell's sum bounds it for 10^6 positive addends of one rounding each (2^-53 each, averaged)."""
import numpy as np
import pytest
import torch

from paper_2512_13965_amd import inputs, transport
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", ["checkerboard", "lattice"])
@pytest.mark.parametrize("n", [255, 256, 257, -1, 0, 1, 255 + 256])
def test_small_and_large_launches_tally_the_same(grid, n):
    binding = require_gpu()
    if n < 255 or n > 300:
        n += 128 * torch.cuda.get_device_properties(0).multi_processor_count
    prob = inputs.checkerboard_problem(8, tau=(0.5, 3.0), src=2) if grid == "checkerboard" else inputs.lattice_problem(16)
    world = binding.World(1 << 17, 1, 1 << 14)
    whole = transport.run_problem(world, prob, n, 3, binding.SAMPLER_MC, chunk=n)
    parts = transport.run_problem(world, prob, n, 3, binding.SAMPLER_MC, chunk=max(1, n // 5))
    world.close()
    np.testing.assert_array_equal(whole["visits"], parts["visits"])
    for k in ("flux", "absorbed", "leak", "cutoff", "wpath", "path"):
        np.testing.assert_allclose(whole[k], parts[k], rtol=1e-12, atol=0.0, err_msg=k)
    assert whole["visits"].sum() == n + whole["transmissions"]
    assert abs(whole["leak"].sum() + whole["absorbed"].sum() + whole["cutoff"].sum() - n) < 1e-9 * n
