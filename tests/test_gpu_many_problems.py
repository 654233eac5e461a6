"""A world of more problems than a workgroup's table of survivor counts has slots (1,024): the counts
per problem are right at every step, and the step takes as long as its particles, not as long as
a search of that table."""
import time

import numpy as np
import pytest

from paper_2512_13965_amd import inputs
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PROB = dict(tau=(0.5, 3.0), src=1)


def _world(binding, problems, hist):
    prob = inputs.checkerboard_problem(4, **PROB)
    world = binding.World(1 << 18, problems, problems * prob.n_cells)
    pids = [world.add_problem(prob, 100 + i) for i in range(problems)]
    for p in pids:
        alive = world.inject(p, 0, hist)
    return world, pids, alive


def _steps(binding, world, alive, each=lambda alive: None):
    """Median time of the steps that begin with 10,000 to 60,000 particles."""
    times = []
    while alive:
        n, t = alive, time.perf_counter()
        alive = world.step(binding.SAMPLER_MC)
        if 10_000 <= n <= 60_000:
            times.append(time.perf_counter() - t)
        each(alive)
    return float(np.median(times))


def test_counts_and_times_of_16384_problems():
    binding = require_gpu()
    few, _, alive = _world(binding, 64, 2048)
    base = _steps(binding, few, alive)
    few.close()
    world, pids, alive = _world(binding, 16_384, 8)
    many = _steps(binding, world, alive)
    for p in pids:                                       # again, with the counts read at every step
        alive = world.inject(p, 8, 8)
    last = {p: world.alive(p) for p in pids}
    assert sum(last.values()) == alive

    def each(alive):
        now = {p: world.alive(p) for p in pids}
        assert sum(now.values()) == alive and all(0 <= now[p] <= last[p] for p in pids)
        last.update(now)

    _steps(binding, world, alive, each)
    for p in (0, 1, 1023, 1024, 9_999, 16_383):
        t = world.tally(p)
        assert abs(t["leak"].sum() + t["absorbed"].sum() + t["cutoff"].sum() - 16) < 1e-10
    world.close()
    print(f"step of 10,000 to 60,000 particles: 64 problems {base * 1e6:.0f} us, 16,384 problems {many * 1e6:.0f} us")
    assert many < 4 * base
