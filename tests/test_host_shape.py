"""Host logic: rows and z segments of the operator's local part, searched at every call.

csrc/apply_shape.hpp (plain C++, what the launch uses) is compiled with g++ and its choice is compared with
the best of every (rows, segments) pair: the same pair on cells of 32 points or more a row with at most
500 planes, where nothing that could win is skipped, and within a tenth in the modelled time on narrow
and long ones.  A call may look at a thousand pairs at most, not at the tens of thousands that a long
narrow cell has (ten nanoseconds each, more than the launch they shape)."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1709_09347_amd", "csrc")
DRIVER = os.path.join(ROOT, "tests", "host", "shape_driver.cpp")


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("shape") / "shape_driver")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
                    "-fno-sanitize-recover=all", "-Wall", "-I", CSRC, DRIVER, "-o", exe], check=True)

    def run(cells):
        txt = "\n".join(" ".join(str(v) for v in c) for c in cells) + "\n"
        r = subprocess.run([exe], input=txt, capture_output=True, text=True, check=True)
        out = [[float(t) for t in line.split()] for line in r.stdout.strip().split("\n")]
        assert len(out) == len(cells)
        return out
    return run


def _cells(seed, n, nx, ny, nz):
    rng = random.Random(seed)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))  # noqa: E731
    out = []
    while len(out) < n:
        p = rng.randint(1, 4)
        c = (log(*nx), log(*ny), max(p, log(*nz)), p, rng.choice([1, 2, 3, 7, 8, 24, 32, 64]), rng.choice([8, 16]))
        if (1 + 2 * p) * c[0] * 32 <= 64 * 1024:   # what a system accepts
            out.append(c)
    return out


def test_ordinary_cells_take_the_best_pair(search):
    cells = _cells(1, 400, (32, 256), (1, 200), (1, 500))
    for c, r in zip(cells, search(cells)):
        assert r[:3] == r[3:6] and r[8] == 1, (c, r)


def test_narrow_and_long_cells_come_close(search):
    cells = _cells(2, 300, (1, 31), (1, 600), (1, 3000)) + [(1, 1, 1, 1, 1, 16), (1, 1, 20000, 4, 1, 16),
                                                            (1, 1500, 1, 1, 64, 8), (256, 1, 1, 1, 1, 16)]
    for c, r in zip(cells, search(cells)):
        assert r[8] == 1 and r[2] <= 1.1 * r[5], (c, r)


@pytest.mark.parametrize("cell", [(5, 96, 48, 1), (8, 96, 48, 2), (16, 64, 200, 1), (4, 256, 512, 1), (8, 512, 512, 1)])
def test_few_pairs_are_looked_at(search, cell):
    for nv in (1, 8, 64):
        r = search([cell + (nv, 16)])[0]
        assert r[6] <= 1200 < r[7], r
