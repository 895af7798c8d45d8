"""The variable coefficient on the multi-iteration path at sides where every
form of it runs: tiles on several lattices one after the other, level 0 on
tiles, residual bands of more than two rows (from 1025 on).

test_iterations: u and the history bit for bit against one launch per iteration.
test_first_restriction: both forms share the residual that restricts to level 1
in the same pass; a cycle from a residual computed alone, whose restriction is a
launch of its own, has to give the same bits.
test_coefficient_set_again: a handle that has solved with another coefficient
against a new one, bit for bit."""
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


@pytest.fixture(scope="module")
def problem(torch_cuda):
    made = {}

    def make(n):
        if n not in made:
            made.clear()
            u0 = np.random.default_rng(n).standard_normal((n, n))  # Dirichlet data on the boundary too
            a, f = W.grf_problem(n, seed=n)
            made[n] = [torch_cuda.from_numpy(v).cuda() for v in (a, f, u0)]
        return made[n]
    return make


@pytest.mark.parametrize("n", [257, 513, 1025, 2049])
@pytest.mark.parametrize("prec,opts", [("fp64", {}), ("fp32", {}), ("bf16", {}), ("fp64", {"max_i": 7, "levels": 4}),
                                       ("bf16", {"max_i": 3})])
def test_iterations(B, torch_cuda, problem, n, prec, opts):
    print("diffusion n=%d %s %s" % (n, prec, opts), flush=True)
    a, f, u0 = problem(n)
    outs = []
    for tb in (2, 0):
        s = B.Solver(2, n, precision=prec, temporal_block=tb, stencil=B.DIFFUSION_5PT_2D, **opts)
        s.set_coefficient(a)
        u = u0.clone()
        r = s.solve_cycles(f, u, 2)
        outs.append((u.cpu().numpy(), r["history"]))
        s.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and outs[0][1] == outs[1][1]


@pytest.mark.parametrize("n", [129, 257, 1025, 2049])
@pytest.mark.parametrize("var", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_first_restriction(B, torch_cuda, problem, n, var, prec):
    torch = torch_cuda
    print("first restriction n=%d var=%s %s" % (n, var, prec), flush=True)
    a, f, u0 = problem(n)
    s = B.Solver(2, n, precision=prec, stencil=B.DIFFUSION_5PT_2D if var else None)
    if var:
        s.set_coefficient(a)
    u = u0.clone()
    s.solve_cycles(f, u, 1)
    r = torch.zeros_like(f)
    s.residual(f, u0, r)
    v = u0.clone()
    s.step_cycle(r, v)
    assert np.array_equal(u.cpu().numpy(), v.cpu().numpy())
    s.close()


@pytest.mark.parametrize("n", [9, 33, 65, 129, 513])
@pytest.mark.parametrize("learned", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "bf16"])
def test_coefficient_set_again(B, torch_cuda, problem, n, learned, prec):
    torch = torch_cuda
    print("coefficient twice n=%d learned=%s %s" % (n, learned, prec), flush=True)
    a, f, u0 = problem(n)
    a2 = torch.exp(-torch.log(a)).contiguous()
    w = torch.from_numpy(LO.jacobi_weights(0.7).astype(np.float32)).cuda()
    outs = []
    for before in ((a,), ()):
        s = B.Solver(2, n, precision=prec, stencil=B.DIFFUSION_5PT_2D)
        for c in before:
            s.set_coefficient(c)
            s.solve_cycles(f, u0.clone(), 2)
        s.set_coefficient(a2)
        if learned:
            s.set_smoother(B.LEARNED, w)
        u = u0.clone()
        r = s.solve_cycles(f, u, 3)
        outs.append((u.cpu().numpy(), r["history"]))
        s.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and outs[0][1] == outs[1][1]
