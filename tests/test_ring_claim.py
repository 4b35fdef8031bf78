"""The serving ring's claim on the CPU: a launch is closed only where no system
is partly claimed, wherever between the workgroup's loads the host publishes a
system and other workgroups take units of it."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2409_15468_amd", "csrc")
CLOSED, NOTHING, AGAIN = -1, -2, -3


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("ring") / "ring_claim")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, os.path.join(HERE, "ring_claim.cpp"), "-o", out], check=True)
    return out


def claim(program, at, claims, leave, idle):
    r = subprocess.run([program] + [str(int(v)) for v in (at, claims, leave, idle)], check=True, capture_output=True, text=True)
    return tuple(int(v) for v in r.stdout.split())


@pytest.mark.parametrize("leave,idle", [(1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("claims", [0, 1, 3, 4])
@pytest.mark.parametrize("at", range(5))
def test_never_closed_inside_a_system(program, at, claims, leave, idle):
    r, split = claim(program, at, claims, leave, idle)
    assert not split
    if 0 < claims < 4 and at == 0:  # part of a system is claimed already: the rest is taken, late or not
        assert r == (7 | claims << 16)


def test_outcomes(program):
    never = 99
    assert claim(program, never, 0, 0, 0) == (NOTHING, 0)
    assert claim(program, never, 0, 1, 0) == (CLOSED, 0)
    assert claim(program, never, 0, 0, 1) == (CLOSED, 0)
    assert claim(program, 0, 0, 0, 0) == (7, 0)       # a system's first unit
    assert claim(program, 0, 0, 1, 0) == (CLOSED, 0)  # not begun: left to the next launch
    assert claim(program, 2, 1, 0, 1) == (AGAIN, 0)   # a claim just before the swap
