"""The learned relaxation's multi-iteration blocks and its one-workgroup
coarse tail (temporal_block=2) against one launch per iteration
(temporal_block=1), which runs the same node arithmetic on other tiles: u, the
residual history and the cycle counts bit for bit, over sides around the block
edges, iteration caps, level counts, schedules, precisions and the constant
coefficient."""
import numpy as np
import pytest

import workloads as W
from oracle import learned as LO

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


def compare(B, torch, n, prec, var, cycles=3, **opts):
    print("learned blocks n=%d %s var=%s %s" % (n, prec, var, opts), flush=True)
    rng = np.random.default_rng(70 + n)
    w = LO.to_bf16(LO.jacobi_weights(0.7) + rng.standard_normal(LO.NW) * 0.01).astype(np.float32)
    u0 = rng.standard_normal((n, n))  # Dirichlet data on the boundary too
    if var:
        a, f = W.grf_problem(n, seed=n)
    else:
        f = W.uniform(2, n, seed=n)
    fd, wd = torch.from_numpy(f).cuda(), torch.from_numpy(w).cuda()
    outs = []
    for tb in (2, 1):
        s = B.Solver(2, n, precision=prec, temporal_block=tb, stencil=B.DIFFUSION_5PT_2D if var else None, **opts)
        if var:
            s.set_coefficient(torch.from_numpy(a).cuda())
        s.set_smoother(B.LEARNED, wd)
        u = torch.from_numpy(u0).cuda()
        r1 = s.solve_cycles(fd, u, cycles)
        v = torch.from_numpy(u0).cuda()
        r2 = s.solve(fd, v, tol=r1["history"][-1] * 1.5, raise_on_status=False)
        acc = torch.zeros((n, n), dtype=torch.float64, device="cuda")
        s.step_cycle(fd, acc)
        outs.append((u.cpu().numpy(), r1["history"], v.cpu().numpy(), r2["cycles"], r2["status"], r2["history"],
                     acc.cpu().numpy()))
        s.close()
    p, q = outs
    for i in (0, 2, 6):
        assert np.array_equal(p[i], q[i], equal_nan=True)
    assert p[1] == q[1] and p[3:6] == q[3:6]


@pytest.mark.parametrize("var", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n", [3, 5, 9, 17, 33, 65, 129, 257, 513])
def test_sides(B, torch_cuda, n, prec, var):
    compare(B, torch_cuda, n, prec, var)


@pytest.mark.parametrize("prec", ["fp64", "bf16"])
@pytest.mark.parametrize("n,opts", [(129, {"max_i": 1}), (129, {"max_i": 2}), (129, {"max_i": 3}), (257, {"max_i": 7}),
                                    (65, {"levels": 1}), (129, {"levels": 2}), (257, {"levels": 3}), (65, {"levels": 3}),
                                    (129, {"levels": 3, "max_i": 5}), (513, {"levels": 4, "max_i": 3}),
                                    (129, {"schedule": [(6, 2), (5, 4), (4, 3), (3, 1), (2, 2), (1, 5), (0, 1)]}),
                                    (129, {"schedule": [(6, 2), (3, 4), (3, 1), (1, 3), (2, 2), (0, 6)]}),
                                    (129, {"schedule": [(6, 2), (5, 4), (4, 3), (3, 3)]})])
def test_options(B, torch_cuda, n, opts, prec):
    compare(B, torch_cuda, n, prec, True, **opts)
