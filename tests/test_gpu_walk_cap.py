"""Walks cut off after 2^24 flights: a walk that never leaves its cell (tau = 10^12, from the middle: its
flights are shorter than the spacing of numbers there) ends with face -2 in a wave of its own (64
lanes on one walk) and among others (lane groups), with the same record bit for bit."""
import math

import numpy as np
import pytest
import torch

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

CAP = 1 << 24


@pytest.mark.parametrize("mode", [0, 1])
def test_walks_that_never_leave_are_cut_off(mode):
    binding = require_gpu()
    # the first 3,100 walks never leave, the others (no material) leave at once: a few of the first to a wave
    n, stuck = 20_000, 3_100
    lt = torch.full((n,), -100.0)
    lt[:stuck] = math.log(1e12)
    half, phi = torch.full((n,), 0.5), torch.arange(n) * 0.1
    host = [lt, torch.ones(n), half, half, torch.cos(phi), torch.sin(phi)]
    cond = binding.DeviceCondInternal(*[t.float().cuda() for t in host])

    def run(first, count):
        sub = binding.DeviceCondInternal(*[v[first:first + count].contiguous() for v in vars(cond).values()])
        ncoll = torch.full((count,), -7, dtype=torch.int32, device="cuda")
        r = binding.mc_transmit_internal(sub, mode, 3, first, ncoll=ncoll).to_host()
        return dict(r, ncoll=ncoll.cpu().numpy())

    many = run(0, n)
    assert (many["face"][:stuck] == -2).all() and (many["ncoll"][:stuck] == CAP).all()
    assert (many["pos"][:stuck] == 0).all()
    np.testing.assert_allclose(many["dir_cos"] ** 2 + many["dir_sin"] ** 2, 1.0, atol=1e-5)
    # a sum of 2^24 flights of 1e-12 in FP32, whose spacing at the sum is 0.9 of a flight: rounding
    # each addition to nearest shifts the mean by up to 3.5 %
    np.testing.assert_allclose(many["path"][:stuck], CAP * 1e-12, rtol=0.1)
    assert (many["face"][stuck:] >= 0).all() and (many["ncoll"][stuck:] == 0).all()
    for i in (0, 1, stuck - 1):
        one = run(i, 1)
        for k in many:
            np.testing.assert_array_equal(one[k], many[k][i:i + 1], err_msg=f"{k} of walk {i}")
