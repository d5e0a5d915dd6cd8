"""The start of a team of workgroups (csrc/team_join.h) in every order in which their accesses can happen: either all
members run, with the same size and places of their own, or none does and exactly one has called the team off."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1701_01170_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("team") / "model")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", f"-I{CSRC}",
                    os.path.join(HERE, "team_join_model.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("more", [0, 1])  # workgroups expected that never register
@pytest.mark.parametrize("polls", [0, 1, 2])
@pytest.mark.parametrize("grid,members", [(1, 1), (2, 2), (3, 1), (3, 2), (3, 3), (4, 2), (4, 3), (4, 4), (4, 0)])
def test_every_interleaving_agrees(model, grid, members, polls, more):
    r = subprocess.run([model, str(grid), str(members), str(polls), str(more)],
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
