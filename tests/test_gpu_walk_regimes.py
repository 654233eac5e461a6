"""The analog walk's two regimes (one lane per walk; a group of lanes per walk once a wave has few
walks left) give the same walks bit for bit: particle i's walk depends on its condition and
stream alone, so a large launch, whose waves run mostly one lane per walk, agrees exactly with
launches of its first n particles, from one walk to a wave (64 lanes on it) upwards."""
import numpy as np
import pytest
import torch

from paper_2512_13965_amd import inputs
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

N = 1 << 18


def _cond(binding, kind):
    if kind == "inside":
        return binding.DeviceCondInternal.from_host(inputs.internal_conditions(N, 5))
    if kind == "xy":
        return binding.DeviceCond.from_host(inputs.xy_conditions(N, 5))
    if kind == "rect":
        return binding.DeviceCond.from_host(inputs.transmission_conditions(N, 5, log_aspect_range=(-1.0, 1.0)))
    tau = {"thin": 0.3, "thick": 60.0, "empty": 0.0}[kind]
    h = inputs.fixed_cell_conditions(N, max(tau, 1e-30), 1.0 if tau else 0.0, 5)
    return binding.DeviceCond.from_host(h)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("kind", ["thin", "thick", "empty", "rect", "xy", "inside"])
def test_walks_do_not_depend_on_the_regime(kind, mode):
    binding = require_gpu()
    cond = _cond(binding, kind)
    walk = binding.mc_transmit_internal if kind == "inside" else binding.mc_transmit

    def run(n):
        ncoll = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        out = binding.DeviceExit.empty(n)
        out.face.fill_(-99)
        r = walk(cond, mode, 11, 1 << 33, ncoll=ncoll, out=out, n=n).to_host()
        r["ncoll"] = ncoll.cpu().numpy()
        return r

    want = run(N)
    assert want["face"].min() >= (-1 if mode == 1 else 0) and want["ncoll"].min() >= 0
    # fewer walks than waves, a few to a wave (granules of 1 to 32 walks), partial granules
    for n in (1, 3, 64, 257, 4097, 6144, 6145, 30_011, 100_003):
        got = run(n)
        for k in want:
            np.testing.assert_array_equal(got[k], want[k][:n], err_msg=f"{k}, {n} walks")
