"""Power-of-two grids: the compact form (marks and ghosts, the one-workgroup
tail) against one whole-grid launch per iteration, bit for bit: every side,
level counts, iteration caps, schedules that revisit, repeat or skip levels,
end on a coarse one, and a non-zero initial guess."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


@pytest.fixture(scope="module")
def B(torch_cuda):
    import paper_1108_2045_amd as P
    return P


@pytest.mark.parametrize("N,opts", [
    (4, {}), (8, {}), (16, {}), (32, {"max_i": 1}), (64, {}), (64, {"levels": 2}), (128, {"max_i": 7}),
    (128, {"levels": 1}), (256, {"levels": 3}), (512, {}), (1024, {"max_i": 3}), (2048, {}),
    (128, {"schedule": [(6, 2), (5, 1), (5, 2), (3, 3), (1, 1), (0, 2)]}),
    (128, {"schedule": [(3, 2), (6, 1), (2, 1), (0, 3), (0, 1), (4, 2), (1, 2)]}),
    (64, {"schedule": [(5, 2), (4, 2), (3, 1), (2, 2)]}),
    (256, {"schedule": [(7, 1), (6, 1), (5, 2), (4, 1), (6, 1), (2, 2), (1, 1), (1, 1), (0, 5)]}),
])
def test_compact_form_is_bitwise_identical(B, torch_cuda, N, opts):
    torch = torch_cuda
    print("pow2 compact N=%d %s" % (N, opts), flush=True)
    rng = np.random.default_rng(N)
    f = torch.from_numpy(W.uniform(2, N, seed=N)).cuda()
    u0 = rng.standard_normal((N, N))
    outs = []
    for tb in (0, 1, 2):
        s = B.Solver(2, N, grid_layout="pow2", temporal_block=tb, **opts)
        u = torch.from_numpy(u0).cuda()
        res = s.solve_cycles(f, u, 3)
        acc = torch.from_numpy(u0).cuda()
        s.step_cycle(f, acc)
        outs.append((u.cpu().numpy(), res["history"], acc.cpu().numpy()))
        s.close()
    for o in outs[1:]:
        assert np.array_equal(o[0], outs[0][0]) and o[1] == outs[0][1] and np.array_equal(o[2], outs[0][2])


@pytest.mark.parametrize("N,opts", [
    (32, {"levels": 2, "max_i": 2}), (64, {"levels": 3, "max_i": 4}), (128, {"levels": 2, "max_i": 5}),
    (256, {"levels": 2, "max_i": 1}), (512, {"levels": 4, "max_i": 3}), (512, {"max_i": 2}), (1024, {"max_i": 6}),
    (1024, {"schedule": [(4, 2), (1, 3), (0, 4)]}), (512, {"schedule": [(2, 2), (0, 2), (1, 1), (0, 7)]}),
    (512, {"schedule": [(3, 2), (1, 4), (1, 2), (0, 1), (0, 2)]}),
])
def test_blocks_of_marks(B, torch_cuda, N, opts):
    """Several iterations per launch on blocks of marks, across the seams of
    the quadrants, and level 0 from level 1's marks, without the one-workgroup
    tail or with few levels in it."""
    test_compact_form_is_bitwise_identical(B, torch_cuda, N, opts)
