"""The one-workgroup kernels (coarse tail, whole solves of small grids)
against the one-launch-per-iteration form, which shares none of their code:
u, the residual history and the cycle counts bit for bit, over sides, level
counts, iteration caps, precisions and the variable coefficient."""
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


def compare(B, torch, d, n, prec, var, cycles=4, **opts):
    print("one-workgroup kernels d=%d n=%d %s var=%s %s" % (d, n, prec, var, opts), flush=True)
    rng = np.random.default_rng(40 + n)
    u0 = rng.standard_normal((n,) * d)  # Dirichlet data on the boundary too
    if var:
        a, f = W.grf_problem(n, seed=n)
    else:
        f = W.uniform(d, n, seed=n)
    fd = torch.from_numpy(f).cuda()
    outs = []
    for tb in (2, 0):
        s = B.Solver(d, n, precision=prec, temporal_block=tb, stencil=B.DIFFUSION_5PT_2D if var else None, **opts)
        if var:
            s.set_coefficient(torch.from_numpy(a).cuda())
        u = torch.from_numpy(u0).cuda()
        r1 = s.solve_cycles(fd, u, cycles)
        v = torch.from_numpy(u0).cuda()
        r2 = s.solve(fd, v, tol=r1["history"][-1] * 1.5, raise_on_status=False)
        outs.append((u.cpu().numpy(), r1["history"], v.cpu().numpy(), r2["cycles"], r2["status"], r2["history"]))
        s.close()
    a2, a0 = outs
    assert np.array_equal(a2[0], a0[0]) and np.array_equal(a2[2], a0[2])
    assert a2[1] == a0[1] and a2[3:] == a0[3:]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("d,n", [(2, 3), (2, 5), (2, 9), (2, 17), (2, 33), (2, 65), (2, 129),
                                 (3, 3), (3, 5), (3, 9), (3, 17), (3, 33)])
def test_laplacian(B, torch_cuda, d, n, prec):
    compare(B, torch_cuda, d, n, prec, False)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n", [3, 5, 17, 33, 65, 129])
def test_variable_coefficient(B, torch_cuda, n, prec):
    compare(B, torch_cuda, 2, n, prec, True)


@pytest.mark.parametrize("prec", ["fp64", "bf16"])
@pytest.mark.parametrize("d,n,opts", [(2, 65, {"levels": 1}), (2, 65, {"levels": 2}), (2, 33, {"levels": 3, "max_i": 1}),
                                      (2, 65, {"max_i": 7}), (2, 129, {"levels": 2}), (2, 129, {"levels": 3, "max_i": 3}),
                                      (3, 17, {"levels": 2, "max_i": 5}), (3, 9, {"levels": 1}),
                                      (3, 33, {"levels": 3, "max_i": 1}),
                                      (2, 65, {"schedule": [(5, 2), (4, 3), (3, 1), (2, 2), (1, 5), (0, 1)]})])
def test_options(B, torch_cuda, d, n, opts, prec):
    compare(B, torch_cuda, d, n, prec, False, **opts)


def test_more_cycles_than_one_launch(B, torch_cuda):
    """A slow schedule (level 0 alone) past the 64 cycles of one launch."""
    compare(B, torch_cuda, 2, 17, "fp64", False, cycles=130, levels=1)


@pytest.mark.parametrize("var", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n,levels", [(65, 2), (65, 4), (65, 5), (129, 3), (129, 4), (129, 5), (129, 6)])
def test_coarsest_side(B, torch_cuda, n, levels, prec, var):
    """The coarsest level at each side the tail writes out (33, 17, 9, 5),
    in FP64 in the reduced-precision cycles."""
    compare(B, torch_cuda, 2, n, prec, var, cycles=3, levels=levels, max_i=5)
