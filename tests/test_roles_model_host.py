"""The wait of the single launch of both kernels' workgroups, on a model device (the kernels' own protocol, compiled for the host): two launches
whose workgroups the XCDs take in opposite orders, and one whose down workgroups come first."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("roles") / "roles_model")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-pthread", "-I", os.path.join(ROOT, "paper_2602_11808_amd", "csrc"),
                           os.path.join(ROOT, "tests", "roles_model.cpp"), "-o", exe])

    def run(may_park, order, seed, limit):
        out = subprocess.run([exe, str(int(may_park)), str(order), str(seed), str(limit)], capture_output=True, text=True, timeout=100, check=True).stdout
        return [dict(zip(("gave_up", "parked", "once", "zero", "early"), map(int, l.split()))) for l in out.splitlines()]
    return run


@pytest.mark.parametrize("order", [1, 2])
def test_a_wait_that_only_waits_can_block_itself(model, order):
    """The fault: with every place taken by down workgroups that wait, nothing ever publishes what they wait for."""
    assert any(l["gave_up"] for l in model(False, order, 1, 20000))


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("seed", range(6))
def test_parking_ends_every_wait(model, order, seed):
    """Nobody gives up, each workgroup's work is done once, after what it needs, and the words are left zero."""
    for l in model(True, order, seed, 1 << 28):
        assert (l["gave_up"], l["once"], l["zero"], l["early"]) == (0, 1, 1, 0), l
        assert l["parked"] < 24 and (order != 2 or l["parked"]), l
