"""Whole solves of small grids run several cycles per launch; how many is bounded
by their iterations, so that a schedule of many iterations does not hold the
GPU in one launch.  Against one launch per iteration: u and the history bit for
bit; the number of launches shows the bound (8192 iterations)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,its,cycles,launches", [
    (17, [450] * 4, 10, (3, 3)),           # 1800 iterations a cycle: four cycles a launch
    (17, [4096, 4094, 1, 1], 3, (3, 3)),   # 8192: one cycle a launch
    (9, [4096, 4096, 1], 3, (4, None)),    # one more: launches of their own
    (17, [2, 4, 4, 4], 100, (2, 2)),       # the default schedule: 64 cycles a launch
])
def test_iterations_per_launch(n, its, cycles, launches):
    import torch
    import paper_1108_2045_amd as P
    print("small solve n=%d %s" % (n, its), flush=True)
    top = len(its) - 1
    sched = [(top - k, it) for k, it in enumerate(its)]
    f = torch.from_numpy(W.uniform(2, n, seed=n)).cuda()
    outs = []
    for tb in (2, 0):
        s = P.Solver(2, n, schedule=sched, temporal_block=tb)
        u = torch.zeros_like(f)
        r = s.solve_cycles(f, u, cycles)
        outs.append((u.cpu().numpy(), r["history"], r["launches"]))
        s.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and outs[0][1] == outs[1][1]
    assert outs[0][2] >= launches[0] and (launches[1] is None or outs[0][2] <= launches[1])
