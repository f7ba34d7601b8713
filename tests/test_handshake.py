"""The marks' protocol of launches whose workgroups wait for each other, on the CPU: csrc/handshake.h, the code that the kernels
run, through every order in which stores and loads may take effect (tests/handshake/interleavings.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def explore(tmp_path_factory):
    exe = os.path.join(str(tmp_path_factory.mktemp("handshake")), "interleavings")
    cmd = ["g++", "-O2", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-D__device__=", "-D__forceinline__=inline",
           "-I" + os.path.join(ROOT, "paper_2508_09072_amd", "csrc"), os.path.join(ROOT, "tests", "handshake", "interleavings.cpp"), "-o", exe]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout

    def run(*args):
        out = subprocess.run([exe] + [str(a) for a in args], stdout=subprocess.PIPE, text=True, timeout=100, check=True).stdout
        return tuple(int(x) for x in out.split())
    return run


@pytest.mark.parametrize("workgroups,looks", [(1, 1), (2, 1), (2, 3), (3, 1)])
def test_whoever_meets_does_the_work_of_those_who_left(explore, workgroups, looks):
    runs, violations = explore("meet", workgroups, 0, looks, 1)
    assert runs >= 1 and violations == 0


@pytest.mark.parametrize("workgroups,keepers,looks", [(1, 1, 2), (2, 1, 2), (1, 2, 2)])
def test_every_keeper_s_work_is_done_once_and_not_too_soon(explore, workgroups, keepers, looks):
    runs, violations = explore("keep", workgroups, keepers, looks, 1)
    assert runs >= 1 and violations == 0


@pytest.mark.parametrize("what,workgroups,keepers", [("meet", 2, 0), ("keep", 1, 1)])
def test_the_exploration_finds_what_a_missing_wait_loses(explore, what, workgroups, keepers):
    # the same code, its waits for its own stores made ineffective by the model
    assert explore(what, workgroups, keepers, 2, 0)[1] > 0


@pytest.mark.parametrize("asked,ticks", [(-1, 3000), (0, 0), (1, 1), (999999, 999999), (1000001, 1000000), (2 ** 29, 1000000),
                                         (2 ** 31 - 2, 1000000)])
def test_no_wait_is_longer_than_ten_milliseconds_a_keeper_s_than_forty(explore, asked, ticks):
    assert explore("ticks", asked) == (ticks, 4 * ticks)
