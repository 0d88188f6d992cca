"""The exchange between workgroups that share a verification walk, stepped through on the host with the kernel's own tags: no
interleaving, however late a member starts and however far the others run ahead, lets a member take another step's sum, or
an earlier replay's, for the one it waits for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("team") / "model")
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2409_10644_amd", "csrc"),
                    os.path.join(ROOT, "tests", "team_protocol_model.cpp"), "-o", exe], check=True)

    def run(members, steps, polls, runs, bits):
        r = subprocess.run([exe, *map(str, (members, steps, polls, runs, bits))], check=True, capture_output=True, text=True)
        words = r.stdout.split()
        return int(words[1]), int(words[3])

    return run


def _bits():
    text = open(os.path.join(ROOT, "paper_2409_10644_amd", "csrc", "team_protocol.h")).read()
    return int(text.split("TEAM_STEP_BITS = ")[1].split(",")[0])


@pytest.mark.parametrize("members,steps,polls,runs", [(2, 10, 1, 2), (2, 12, 2, 3), (3, 6, 1, 2), (3, 8, 0, 2), (4, 3, 0, 1)])
def test_no_interleaving_mistakes_one_message_for_another(model, members, steps, polls, runs):
    states, wrong = model(members, steps, polls, runs, _bits())
    assert states > 500 and wrong == 0


def test_two_bits_of_the_step_are_not_enough(model):
    """Steps s and s + 4 look the same then: a member that starts late takes what one that runs ahead alone has published."""
    assert model(2, 7, 1, 1, 2)[1] > 0


def test_every_step_of_the_largest_tree_has_a_number():
    """A path meets one context per level, which rejects at most as many candidates as the level's branching factor.  For given
    factors the tree with the fewest nodes has them in ascending order, so ones come first."""
    best = 0

    def grow(least, width, nodes, total, levels):
        nonlocal best
        best = max(best, total + min(32 - levels, 4096 - nodes))        # levels of one child each in front
        if levels == 32:
            return
        for b in range(least, 65):
            if nodes + width * b > 4096:
                break
            grow(b, width * b, nodes + width * b, total + b, levels + 1)

    grow(2, 1, 0, 0, 0)
    steps = best + 1                            # and the sum of the distribution that the walk ends in
    assert steps == 157 and steps < 1 << _bits()
