"""Tallies read a few columns at a time are those read all at once, bit for bit, and obey the
tallies' own relations, for grids on both sides of the number of cells that one pass of the
read-out holds (524,288 doubles: 131,072 cells of four columns, 104,857 of five, all of one)."""
import ctypes

import numpy as np
import pytest

from paper_2512_13965_amd import inputs
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

A = ("flux", "absorbed", "leak", "cutoff")
B = ("wpath", "path", "visits", "rejected_w", "rejected_n")


@pytest.mark.parametrize("n", [1, 16, 323, 324, 362, 363, 724, 725])
def test_columns_do_not_depend_on_how_they_are_read(n):
    binding = require_gpu()
    world = binding.World(1 << 16, 2, 2 * n * n)
    world.add_problem(inputs.checkerboard_problem(n, src=1), 9)         # the second one's cells start behind it
    prob = inputs.random_problem(n, side_range=(n, n))[0]
    assert prob.n_cells == n * n
    pid = world.add_problem(prob, 3)
    alive = world.inject(pid, 0, 20_000)
    while alive:
        alive = world.step(binding.SAMPLER_MC)
    whole = world.tally(pid)
    L, h, s = world._L, world._h, binding._stream()
    for call, names in ((L.gmc_problem_tally, A), (L.gmc_problem_path_tally, B)):
        for want in [(k,) for k in names] + [names[1:3], names[::2]]:
            out = {k: np.full(n * n, -1.0) for k in want}
            args = [out[k].ctypes.data if k in out else None for k in names]
            assert call(h, pid, *args, s) == binding.GMC_OK
            for k in want:
                np.testing.assert_array_equal(out[k], whole[k], err_msg=f"{k} of {want}")
        assert call(h, pid, *[None] * len(names), s) == binding.GMC_OK
    tau, c = np.asarray(prob.tau, np.float64).ravel(), np.asarray(prob.c, np.float64).ravel()
    siga, V = (1.0 - c) * tau / prob.L, prob.L * prob.L
    flux = np.where(siga > 0, whole["absorbed"] / (V * np.where(siga > 0, siga, 1.0)), whole["wpath"] / V)
    np.testing.assert_array_equal(whole["flux"], flux)                  # the same IEEE operations
    assert whole["visits"].sum() == 20_000 + world.transmissions()
    world.close()
