"""Width-128 transport steps of more samples than the sampler's waves hold at once (twelve waves of 32
samples to a compute unit), so that waves go on to a second tile: captured steps against
direct ones, and against a bank so small that no wave does."""
import numpy as np
import pytest
import torch

from paper_2512_13965_amd import inputs, transport
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["bf16", "fp8"])
def test_captured_steps_whose_waves_take_several_tiles(precision):
    binding = require_gpu()
    once = 32 * 12 * torch.cuda.get_device_properties(0).multi_processor_count
    prob = inputs.homogeneous_problem(32, 0.5, 0.9, True)          # reflecting: all birth cells, none leaks
    model = binding.Model(inputs.pack_blob(inputs.random_weights(128, 3)), precision)
    n = 5 * once // 2
    runs = {}
    for label, graphs, chunk in (("graph", True, n), ("direct", False, n), ("small", False, once // 4)):
        world = binding.World(n, 1, 1 << 11)
        world.set_graphs(graphs)
        pid = world.add_problem(prob, 8)
        alive = steps = over = injected = 0
        while injected < n or alive:
            if injected < n and alive + min(chunk, n - injected) <= (n if chunk == n else once // 2):
                count = min(chunk, n - injected)
                alive = world.inject(pid, injected, count)
                injected += count
            over += alive > once
            alive = world.step(binding.SAMPLER_GMC, model, 2)
            steps += 1
        runs[label] = dict(world.tally(pid), transmissions=world.transmissions())
        assert (over > 1) == (chunk == n), (label, over)
        world.close()
    model.close()
    for label in ("graph", "small"):
        assert runs[label]["transmissions"] == runs["direct"]["transmissions"]
        for k in ("flux", "absorbed", "leak", "cutoff", "wpath", "path", "visits"):
            np.testing.assert_allclose(runs[label][k], runs["direct"][k], rtol=1e-12, atol=1e-12 * n, err_msg=f"{label} {k}")
