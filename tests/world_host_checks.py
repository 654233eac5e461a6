"""Host side of the transport world against a stand-in for the HIP runtime (tests/hip_stub.cpp):
what it launches and copies, and what it does after a call that failed.  Run by
tests/test_world_cpu.py in a child process with the stand-in preloaded:
`python -m tests.world_host_checks <library> <stub> <check>`."""
import ctypes
import sys

import numpy as np

from paper_2512_13965_amd import inputs

P, I32, I64, U64, I = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_uint64, ctypes.c_int
OK, EDEVICE, MC = 0, -3, 1


class Desc(ctypes.Structure):
    _fields_ = [("nx", I32), ("ny", I32), ("L", ctypes.c_double), ("tau", P), ("c", P), ("src_x0", I32),
                ("src_y0", I32), ("src_nx", I32), ("src_ny", I32), ("reflect", I32), ("w_min", ctypes.c_double),
                ("seed", U64), ("src_face", I32), ("Ly", ctypes.c_double), ("xy", I32), ("max_visits", I64)]


class Stub:
    def __init__(self, path):
        S = ctypes.CDLL(path)
        S.stub_watch.argtypes = [ctypes.c_char_p, I]
        S.stub_name.restype = ctypes.c_char_p
        S.stub_grid.restype = S.stub_block.restype = ctypes.c_uint32
        S.stub_arg.restype = S.stub_restored_word.restype = U64
        S.stub_copied.restype = S.stub_pinned.restype = I64
        self.S = S

    def counts(self, *v):
        self.S.stub_counts((U64 * len(v))(*v), len(v))

    def restored(self):
        return [self.S.stub_restored_word(i) for i in range(self.S.stub_restored())]

    def launches(self, name):
        S = self.S
        return [i for i in range(S.stub_launches()) if name in S.stub_name(i).decode()]


class World:
    """The C entry points of one world."""

    def __init__(self, lib, cap, problems, cells):
        L = ctypes.CDLL(lib)
        L.gmc_world_create.argtypes = [I64, I32, I64, P]
        L.gmc_world_destroy.argtypes = [P]
        L.gmc_problem_add.argtypes = [P, P, P, P]
        L.gmc_world_inject.argtypes = [P, I32, U64, I64, P, P]
        L.gmc_transport_step.argtypes = [P, I, P, I, P, P]
        L.gmc_problem_alive.argtypes = [P, I32, P]
        L.gmc_problem_tally.argtypes = [P, I32, P, P, P, P, P]
        L.gmc_problem_path_tally.argtypes = [P, I32, P, P, P, P, P, P]
        L.gmc_world_transmissions.argtypes = [P, P]
        self.L, self.h = L, P()
        assert L.gmc_world_create(cap, problems, cells, ctypes.byref(self.h)) == OK

    def add(self, prob):
        tau, c = np.ascontiguousarray(prob.tau, np.float64), np.ascontiguousarray(prob.c, np.float64)
        d = Desc(prob.nx, prob.ny, prob.L, tau.ctypes.data, c.ctypes.data, prob.src_x0, prob.src_y0, prob.src_nx,
                 prob.src_ny, int(prob.reflect), prob.w_min, 1, -1, 0.0, 0, 0)
        pid = I32()
        assert self.L.gmc_problem_add(self.h, ctypes.byref(d), ctypes.byref(pid), None) == OK
        return pid.value

    def inject(self, pid, h, n):
        a = I64()
        return self.L.gmc_world_inject(self.h, pid, h, n, None, ctypes.byref(a)), a.value

    def step(self):
        a = I64()
        return self.L.gmc_transport_step(self.h, MC, None, 0, None, ctypes.byref(a)), a.value

    def alive(self, pid):
        a = I64()
        assert self.L.gmc_problem_alive(self.h, pid, ctypes.byref(a)) == OK
        return a.value

    def transmissions(self):
        a = I64()
        assert self.L.gmc_world_transmissions(self.h, ctypes.byref(a)) == OK
        return a.value


def failed_calls(lib, stub):
    """A step or an injection whose wait fails leaves the world as it was: the next call works on
    the same bank, with the counts of all particles and of each problem before the failure."""
    S = stub.S
    S.stub_watch(b"12apply_kernel", 0)           # the bank a step reads
    w = World(lib, 1 << 10, 2, 256)
    prob = inputs.checkerboard_problem(8, src=2)
    a, b = w.add(prob), w.add(prob)
    stub.counts(70, 70, 0)
    assert w.inject(a, 0, 100) == (OK, 70)
    stub.counts(90, 70, 20)
    assert w.inject(b, 0, 30) == (OK, 90)

    def state():
        return w.alive(a), w.alive(b), w.transmissions()

    def failing(call):
        S.stub_clear()
        S.stub_fail_syncs(1 << 30)
        assert call()[0] == EDEVICE
        S.stub_fail_syncs(0)

    # a step that failed once its counters were stored
    stub.counts(50, 40, 10)
    failing(w.step)
    bank = S.stub_arg(stub.launches("12apply_kernel")[0], 0)
    assert state() == (70, 20, 0)
    S.stub_clear()
    stub.counts(60, 45, 15)
    assert w.step() == (OK, 60)
    assert stub.restored() == [90, 70, 20] and stub.launches("reset_kernel")[0] == 0
    assert S.stub_arg(stub.launches("12apply_kernel")[0], 0) == bank
    assert state() == (45, 15, 90)
    # an injection that failed after its births were counted
    stub.counts(160, 145, 15)
    failing(lambda: w.inject(a, 100, 100))
    assert state() == (45, 15, 90)
    S.stub_clear()
    stub.counts(80, 65, 15)
    assert w.inject(a, 100, 20) == (OK, 80)
    assert stub.restored() == [60, 45, 15] and stub.launches("reset_kernel")[0] == 0
    # undisturbed calls: no repair, the other bank
    S.stub_clear()
    assert w.step() == (OK, 80)
    assert S.stub_arg(stub.launches("12apply_kernel")[0], 0) != bank and not stub.launches("reset_kernel")


def tally_bytes(lib, stub):
    """Reading tallies brings back the columns asked for and nothing else."""
    w = World(lib, 1 << 10, 1, 1 << 20)
    prob = inputs.checkerboard_problem(500, src=2)
    pid, n = w.add(prob), prob.n_cells
    out = [np.zeros(n) for _ in range(5)]
    at = [o.ctypes.data for o in out]
    for call, args in ((w.L.gmc_problem_tally, (at[0], None, None, None)),
                       (w.L.gmc_problem_tally, (None, at[1], None, at[3])),
                       (w.L.gmc_problem_tally, tuple(at[:4])),
                       (w.L.gmc_problem_path_tally, (None, None, at[2], None, None)),
                       (w.L.gmc_problem_path_tally, tuple(at))):
        stub.S.stub_clear()
        assert call(w.h, pid, *args, None) == OK
        assert stub.S.stub_copied(2) <= 8 * n * sum(a is not None for a in args), args


def add_bytes(lib, stub):
    """Adding a problem uploads its two FP64 materials and ln tau in FP32, and its description."""
    w = World(lib, 1 << 10, 1, 1 << 20)
    prob = inputs.checkerboard_problem(500, src=2)
    stub.S.stub_clear()
    w.add(prob)
    assert stub.S.stub_copied(1) <= (8 + 8 + 4) * prob.n_cells + 1024


def finish_grid(lib, stub):
    """The kernel that ends a step has a thread for every counter of the world."""
    for problems in (1, 255, 256, 65536):
        w = World(lib, 1 << 10, problems, 256)
        pid = w.add(inputs.checkerboard_problem(8, src=2))
        stub.S.stub_clear()
        stub.counts(5, *[5 if p == pid else 0 for p in range(problems)])
        assert w.inject(pid, 0, 10) == (OK, 5)
        i, = stub.launches("finish_kernel")
        threads = stub.S.stub_grid(i) * stub.S.stub_block(i)
        assert 1 + problems <= threads < 1 + problems + 256, (problems, threads)
        assert w.L.gmc_world_destroy(w.h) == OK


def one_problem(lib, stub):
    """A step of a world with one problem takes that problem's key and shape from the launch, one of
    a world with several reads each particle's; problems may come and go in any order."""
    w = World(lib, 1 << 10, 300, 300 * 64)
    prob = inputs.checkerboard_problem(8, src=2)
    w.L.gmc_problem_remove.argtypes = [P, I32]
    held = []

    def keyed(pid):
        stub.S.stub_clear()
        stub.counts(5, *[5 if p == pid else 0 for p in range(300)])
        assert w.inject(pid, 0, 10) == (OK, 5)
        stub.counts(0)
        assert w.step() == (OK, 0)
        name = stub.S.stub_name(stub.launches("walk_step_kernel")[0]).decode()
        assert "Lb0ELb0E" in name or "Lb0ELb1E" in name, name
        return "Lb0ELb1E" in name

    rng = np.random.default_rng(1)
    for _ in range(60):
        if held and (len(held) == 4 or rng.random() < 0.5):
            assert w.L.gmc_problem_remove(w.h, held.pop(rng.integers(len(held)))) == OK
        else:
            held.append(w.add(prob))
        if held:
            assert keyed(held[-1]) == (len(held) > 1), held


def small_tallies(lib, stub):
    """Few particles are tallied by workgroups of at most 256 of them, many by at most one workgroup
    to a compute unit (256 of them here); every particle has a thread either way."""
    w = World(lib, 1 << 20, 1, 256)
    pid = w.add(inputs.checkerboard_problem(8, src=2))
    h = 0
    for n in (1, 256, 257, 4000, 128 * 256, 128 * 256 + 1, 500_000):
        stub.S.stub_clear()
        stub.counts(n, n)
        assert w.inject(pid, h, n) == (OK, n)
        stub.counts(0)
        assert w.step() == (OK, 0)
        h += n
        for i in stub.launches("apply_kernel"):                 # the births' and the step's
            grid, block = stub.S.stub_grid(i), stub.S.stub_block(i)
            if n <= 128 * 256:
                assert block == 256 and grid == (n + 255) // 256, (n, grid, block)
            else:
                assert block == 1024 and grid == min((n + 1023) // 1024, 256), (n, grid, block)


def main():
    lib, stub, check = sys.argv[1:4]
    globals()[check](lib, Stub(stub))
    print("OK")


if __name__ == "__main__":
    main()
