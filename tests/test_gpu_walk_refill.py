"""Lanes that take several walks in turn: a launch of three walks and more to every lane that the
walk's grid can hold (6 workgroups of 256 lanes to a compute unit) against launches of its
first and its last walks so small that no lane ever takes a second one, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2512_13965_amd import inputs
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def _cond(binding, kind, n):
    if kind == "inside":
        return binding.DeviceCondInternal.from_host(inputs.internal_conditions(n, 5))
    if kind == "xy":
        return binding.DeviceCond.from_host(inputs.xy_conditions(n, 5))
    if kind == "rect":
        return binding.DeviceCond.from_host(inputs.transmission_conditions(n, 5, log_aspect_range=(-1.0, 1.0)))
    if kind == "mixed":
        return binding.DeviceCond.from_host(inputs.transmission_conditions(n, 5))
    return binding.DeviceCond.from_host(inputs.fixed_cell_conditions(n, {"thin": 0.3, "thick": 60.0}[kind], 0.98, 5))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("kind", ["thin", "thick", "mixed", "rect", "xy", "inside"])
def test_refilled_lanes_walk_the_same(kind, mode):
    binding = require_gpu()
    lanes = torch.cuda.get_device_properties(0).multi_processor_count * 6 * 256
    n = 3 * lanes + 77
    cond = _cond(binding, kind, n)
    walk = binding.mc_transmit_internal if kind == "inside" else binding.mc_transmit

    def run(first, count):
        sub = type(cond)(*[None if v is None else v[first:first + count].contiguous() for v in vars(cond).values()])
        ncoll = torch.full((count,), -7, dtype=torch.int32, device="cuda")
        out = binding.DeviceExit.empty(count)
        out.face.fill_(-99)
        r = walk(sub, mode, 11, (1 << 33) + first, ncoll=ncoll, out=out).to_host()
        return dict(r, ncoll=ncoll.cpu().numpy())

    want = run(0, n)
    assert want["face"].min() >= (-1 if mode == 1 else 0) and want["ncoll"].min() >= 0
    for count in (4_097, 30_011, 100_003):
        for first in (0, n // 2, n - count):
            got = run(first, count)
            for k in want:
                np.testing.assert_array_equal(got[k], want[k][first:first + count], err_msg=f"{k}, {count} from {first}")
