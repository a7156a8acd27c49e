"""Host logic: how many energies' Hankel SVDs run side by side in a batched solve.

csrc/groups.hpp (plain C++, the rule that the extraction uses) is compiled with g++: groups of up to 32 energies
and 64 MiB of moments where there is memory, and never more than a quarter of the budget that the batch
was sized by, past the one energy that a solve needs anyway."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_groups_fit_beside_the_batch(tmp_path):
    exe = str(tmp_path / "groups_driver")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
                    "-I", os.path.join(ROOT, "paper_1709_09347_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "groups_driver.cpp"), "-o", exe], check=True)
    cases = [(ne, mom, n, budget) for ne in (1, 7, 32, 200) for mom in (0.0, 1.6e6, 3.0e8) for n in (1, 64, 256)
             for budget in (1.0, 1e6, 2e7, 4e8, 1.7e11)]
    out = subprocess.run([exe], input="\n".join("%d %r %d %r" % c for c in cases), capture_output=True, text=True, check=True)
    rows = [line.split() for line in out.stdout.strip().split("\n")]
    for (ne, mom, n, budget), (g, held) in zip(cases, rows):
        g, held = int(g), float(held)
        assert 1 <= g <= min(ne, 32) and (g == 1 or held <= 0.25 * budget) and (g == 1 or g * mom <= 64 * 2 ** 20)
        if budget == 1.7e11:   # most of a card: as many as the moments allow
            assert g == max(1, min(ne, 32, int(64 * 2 ** 20 / max(mom, 1.0))))
