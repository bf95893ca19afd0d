"""Waits of the recurrent kernels that take a chunk of time steps per launch, on the CPU: the header that they share."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2007_10412_amd", "csrc")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rnn") / "rnn_chunk_probe")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + CSRC, os.path.join(HERE, "rnn_chunk_probe.cpp"), "-o", exe])
    return lambda *args: [[int(v) for v in line.split()]
                          for line in subprocess.check_output([exe] + list(args), text=True).splitlines()]


def test_bounds_of_two_contexts_differ(probe):
    """Of two launches that each hold a part of an XCD one has to give way first, whatever the lengths of their models."""
    by_own = {}
    for chunk, own, bound in probe():
        by_own.setdefault(own, set()).add(bound)
        assert max(2048, 64 * (chunk - 16)) <= bound - 256 * own <= max(2048, 64 * (chunk + 16))
    for a in by_own:
        for b in by_own:
            assert a == b or min(abs(u - v) for u in by_own[a] for v in by_own[b]) >= 256


def test_launches_that_do_not_try(probe):
    """About the same time steps go to the stand-in whatever the chunk: 0, 32, 96, 224 and 480 after failures in a row."""
    for chunk, fails, skip in probe("skip"):
        steps = 32 * (2 ** min(fails, 4) - 1)
        if chunk <= 32:
            assert 32 * skip == steps
        else:
            assert abs(skip * chunk - steps) <= chunk / 2, (chunk, fails, skip)
