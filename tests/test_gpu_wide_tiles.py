"""Tiles of 32, 64 and 96 samples against full ones, bit for bit: launches whose samples per compute
unit lie at the edges of a tile size, and remainders of such sizes behind full rounds.  A launch that
asks for the raw states takes full tiles beyond 96 samples per compute unit, and is the reference."""
import numpy as np
import pytest
import torch

from paper_2512_13965_amd import inputs
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("net,precision,hidden", [("mlp", "bf16", 512), ("mlp", "fp8", 512), ("mlp", "bf16", 256),
                                                  ("mlp", "fp32", 256), ("mlp", "fp32", 128),
                                                  ("mlp", "fp8", 256), ("film", "bf16", 512), ("film", "bf16", 256)])
@pytest.mark.parametrize("integrator", ["euler", "rk4"])
def test_tile_sizes_agree(net, precision, hidden, integrator):
    binding = require_gpu()
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    full = 128 * cu
    w = inputs.random_weights(hidden, 3) if net == "mlp" else inputs.random_film_weights(hidden, 3)
    m = binding.Model(inputs.pack_blob(w), precision)
    N = full + 100 * cu
    cond = binding.DeviceCond.from_host(inputs.transmission_conditions(N, 8))
    raw = torch.empty(5, N, device="cuda")
    want = binding.gmc_sample(m, cond, integrator, 2, 6, 0, raw=raw).to_host()
    assert torch.isfinite(raw).all()
    sizes = [1, 31, 33, 32 * cu, 32 * cu + 1, 64 * cu, 64 * cu + 1, 78 * cu + 33, 96 * cu, 96 * cu + 1, full, full + 5,
             full + 64 * cu + 1, full + 96 * cu, full + 96 * cu + 1]
    for n in sizes:
        got = binding.gmc_sample(m, cond, integrator, 2, 6, 0, n=n).to_host()
        for k in want:
            np.testing.assert_array_equal(got[k], want[k][:n], err_msg=f"{k}, {n} samples")
    m.close()
