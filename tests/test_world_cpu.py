"""CPU checks of the transport world's host code against a stand-in for the HIP runtime
(tests/hip_stub.cpp, tests/world_host_checks.py), one child process each."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC",
                           os.path.join(ROOT, "tests", "hip_stub.cpp"), "-o", out])
    return out


def _check(stub, name):
    from paper_2512_13965_amd import binding
    preload = " ".join([stub, *os.environ.get("LD_PRELOAD", "").split()])
    r = subprocess.run([sys.executable, "-m", "tests.world_host_checks", binding.LIB_PATH, stub, name], cwd=ROOT,
                       env=dict(os.environ, LD_PRELOAD=preload), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout + r.stderr


def test_failed_calls_leave_the_world_as_it_was(stub):
    _check(stub, "failed_calls")


def test_tallies_are_read_by_the_columns_asked_for(stub):
    _check(stub, "tally_bytes")


def test_adding_a_problem_uploads_its_materials_once(stub):
    _check(stub, "add_bytes")


def test_the_end_of_a_step_has_a_thread_for_every_counter(stub):
    _check(stub, "finish_grid")


def test_the_one_problem_of_a_world_is_known(stub):
    _check(stub, "one_problem")


def test_few_particles_are_tallied_by_small_workgroups(stub):
    _check(stub, "small_tallies")
