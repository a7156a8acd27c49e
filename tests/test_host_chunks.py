"""Host logic: the chunks of the residual update and the buffers of their partial sums.

The tuner times the update in chunks of three lengths on one buffer; a solve shortens the tuned
length for small batches and sizes its own buffer.  csrc/chunks.hpp (plain C++, the rules that the
launches use) is compiled with g++: over every cell size the last partial sum of every trial lies
inside the buffer, and the chunks cover the cell."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1709_09347_amd", "csrc")
DRIVER = os.path.join(ROOT, "tests", "host", "chunks_driver.cpp")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("chunks") / "chunks_driver")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
                    "-fno-sanitize-recover=all", "-Wall", "-I", CSRC, DRIVER, "-o", exe], check=True)
    return exe


# the tuner's batch is 256 runs on cells up to 52,000 complex128 points, at least 8
@pytest.mark.parametrize("runs", [1, 8, 30, 255, 256])
def test_trials_stay_inside_their_buffer(driver, runs):
    r = subprocess.run([driver, "1", "80000", str(runs)], capture_output=True, text=True, check=True)
    lines = r.stdout.split("\n")
    assert lines[:-2] == [], lines[:5]
    assert lines[-2] == "checked 240000"
