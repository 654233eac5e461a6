"""Tallies and survivor counts of workgroups that take several tiles of particles: the same
histories whatever the launch's size (edges of a 1,024-particle tile, one tile to a workgroup,
several), and whatever other problems share the bank (more of them than one table of cells
holds).  Tallies of the same histories differ by the order of FP64 additions only: 1e-12 of the
cell's sum bounds it for 10^6 positive addends of one rounding each (2^-53 each, averaged)."""
import numpy as np
import pytest

from paper_2512_13965_amd import inputs, transport
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

KEYS = ("flux", "absorbed", "leak", "cutoff", "wpath", "path")


def _same(a, b, label):
    np.testing.assert_array_equal(a["visits"], b["visits"], err_msg=label)
    for k in KEYS:
        np.testing.assert_allclose(a[k], b[k], rtol=1e-12, atol=0.0, err_msg=f"{label} {k}")


@pytest.mark.parametrize("n", [1, 511, 512, 513, 1023, 1025, 400_001])
def test_chunks_of_any_size_tally_the_same(n):
    binding = require_gpu()
    prob = inputs.checkerboard_problem(8, tau=(0.5, 3.0), src=2)
    world = binding.World(1 << 19, 1, 1 << 12)
    whole = transport.run_problem(world, prob, n, 3, binding.SAMPLER_MC, chunk=n)
    parts = transport.run_problem(world, prob, n, 3, binding.SAMPLER_MC, chunk=max(1, n // 7))
    world.close()
    _same(whole, parts, f"{n} histories")
    assert whole["visits"].sum() == n + whole["transmissions"]
    assert abs(whole["leak"].sum() + whole["absorbed"].sum() + whole["cutoff"].sum() - n) < 1e-9 * n


def test_many_problems_share_workgroups():
    # 600 problems of 5 to 9 histories each: a workgroup's tile holds many problems, and their
    # 600 * 25 cells overflow its table of 4,096
    binding = require_gpu()
    P, prob = 600, inputs.checkerboard_problem(5, tau=(0.5, 3.0), src=1)
    hist = [5 + i % 5 for i in range(P)]
    world = binding.World(1 << 14, P, P * prob.n_cells)
    pids = [world.add_problem(prob, 100 + i) for i in range(P)]
    for i, pid in enumerate(pids):
        alive = world.inject(pid, 0, hist[i])
    while alive:
        alive = world.step(binding.SAMPLER_MC)
        assert sum(world.alive(p) for p in pids) == alive
    got = [world.tally(p) for p in pids]
    world.close()
    alone = binding.World(1 << 10, 1, 1 << 10)
    for i in (0, 1, 17, 299, 598, 599):
        want = transport.run_problem(alone, prob, hist[i], 100 + i, binding.SAMPLER_MC)
        _same(got[i], want, f"problem {i}")
    alone.close()


@pytest.mark.parametrize("n", [3, 700, 200_001])
def test_streaming_refills_lanes(n):
    # the first-flight split's streaming kernel: fewer particles than waves, than lanes, and more
    # than its lanes at once (256 CUs of 512); with one crossing per step, with many, and with a
    # second problem in the world (its kernel then reads each particle's problem)
    binding = require_gpu()
    prob = inputs.lattice_problem(4)
    w = inputs.random_weights(128, 7, flags=2)
    m = binding.Model(inputs.pack_blob(w), "bf16")
    runs = {}
    for label, streaming, second in (("one", 1, False), ("many", 64, False), ("two problems", 64, True)):
        world = binding.World(1 << 18, 2, 1 << 12)
        if second:
            world.add_problem(inputs.checkerboard_problem(4, src=1), 1)
        runs[label] = transport.run_problem(world, prob, n, 5, binding.SAMPLER_GMC, m, 2, streaming=streaming)
        world.close()
    m.close()
    for label in ("many", "two problems"):
        _same(runs["one"], runs[label], label)
        assert runs[label]["transmissions"] == runs["one"]["transmissions"]
    assert runs["many"]["steps"] < runs["one"]["steps"]
