"""The tile tuner times what a full batch runs: both launches of a pair of iterations, the one that leaves
x alone and the one that adds two directions to it, and keeps the height of the least sum.

Tolerance: the log prints times to 1e-4 ms, so the printed sums of the choice and of the best differ
by at most two units of that."""
import re

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_height_is_the_least_sum_of_both_launches(cuda):
    import torch
    import paper_1709_09347_amd as cbs
    sysw = W.make_system(24, 20, 15, 0.4, 6, 5, 721, 722, with_proj=True, r_c=1.1)
    s = cbs.System.from_workload(sysw)
    assert s.tiling()[2] == ""
    s.bicg(0.3, [2.0 + 0.5j], torch.from_numpy(W.make_rhs(sysw.n, 1, 723)).to(cuda), cbs.default_params(max_iter=2))
    torch.cuda.synchronize()
    ty64, ty32, log = s.tiling()
    print(log, flush=True)
    for tag, ty in (("c128", ty64), ("c64", ty32)):
        rows = re.findall(tag + r" ty=(\d+) ([\d.]+) \+ ([\d.]+) ms", log)
        assert [int(r[0]) for r in rows] == list(range(1, len(rows) + 1)) and len(rows) > 1
        total = {int(r[0]): float(r[1]) + float(r[2]) for r in rows}
        assert total[ty] <= min(total.values()) + 2.1e-4
