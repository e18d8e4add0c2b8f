"""The claims of the light PP tiles' items (csrc/light_claims.hpp), walked on the host:
every item exactly once, whatever the number of light tiles and the order of the waves.

Workgroups and waves of the four launches (force beside PM and PP alone, the adjoint
beside PM and alone), of grids that are no multiple of the 8 groups and of a grid of
fewer.  The numbers of light tiles are all around the steps at which items begin to come
from counters and the chunks of a claim grow, and strides through the rest."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    exe = str(tmp_path_factory.mktemp("claims") / "walk")
    subprocess.run([cxx, "-O2", "-std=c++17", "-o", exe, os.path.join(HERE, "light_claims_walk.cpp")], check=True)
    return exe


@pytest.mark.parametrize("grid,waves", [(384, 8), (512, 8), (160, 9), (256, 9), (204, 8), (133, 9), (5, 8)])
@pytest.mark.parametrize("per", [4, 8])
def test_every_item_once(walk, grid, waves, per):
    ranges = [(0, 40, 1), (41, 10000, 97)]
    nw = grid * waves
    for items in (4 * nw, 6 * nw, 8 * nw):      # fixed / not, chunks of 2 / 3 and of 3 / 4
        n = items // per
        ranges.append((max(n - 20, 0), n + 20, 1))
    for seed, (a, b, step) in enumerate(ranges):
        r = subprocess.run([walk] + [str(v) for v in (grid, waves, per, a, b, step, seed)],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stdout
