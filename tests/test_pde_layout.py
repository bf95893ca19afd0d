"""Step counts and runs of the reaction-diffusion kernels, on the CPU: the header that entry points, launch and kernels share."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2007_10412_amd", "csrc")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pde") / "pde_layout_probe")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + CSRC, os.path.join(HERE, "pde_layout_probe.cpp"), "-o", exe])

    def run(*args):
        out = subprocess.check_output([exe] + [str(a) for a in args], text=True)
        return [[int(v) for v in line.split()] for line in out.splitlines()]
    return run


def test_pairs_of_steps_end(probe):
    """Up to 2^32 - 2 steps (one interior cell): the loop over pairs ends less than two steps before the end."""
    counts = [1, 2, 3, 4, 5, 40960, 40961, 2 ** 31 - 1, 2 ** 31, 2 ** 32 - 5, 2 ** 32 - 4, 2 ** 32 - 3, 2 ** 32 - 2]
    for steps, turns, t in probe(*counts):
        assert turns <= 2 and 0 <= steps - t < 2, (steps, turns, t)


def test_runs_fit_the_workspace(probe):
    """The sampling waves' runs do not overlap, hold every entry at fraction 1 and fit what rad_pde_workspace_bytes asks for."""
    for cells, steps, ppm, entries, wrong, room in probe("runs"):
        assert not wrong and entries <= room, (cells, steps, ppm)
        assert entries <= cells * (steps + 1) and entries >= cells * (steps + 1) * ppm // 1000000
        if ppm == 1000000:
            assert entries == cells * (steps + 1)
