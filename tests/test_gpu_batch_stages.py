"""The batched solver's stage lists against single solves: sides at which the
stages change (65 | 129: one workgroup or stages; 257 | 513: one or several
restriction steps), small and large batches (latency or throughput form of
the passes), iteration caps whose levels take several passes, initial guesses
with boundary data, and solves past the cycles of one launch: u and the cycle
counts bit for bit, the norms to the rounding of their summation order."""
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


@pytest.mark.parametrize("sides,prec,opts", [
    ([3, 5, 65, 129, 257, 513, 1025], "fp64", {}),
    ([3, 5, 9, 17, 33, 65, 129, 129, 1025, 257], "bf16", {"max_i": 7}),
    ([2049, 65, 129], "fp32", {"max_i": 3}),
    ([1025, 1025, 1025, 513, 257, 129], "fp32", {"max_i": 6}),
    ([129] * 20 + [65] * 5, "fp64", {"max_i": 1}),
])
def test_batch_equals_single_solves(B, torch_cuda, sides, prec, opts):
    torch = torch_cuda
    print("batch stages %s %s %s" % (sides, prec, opts), flush=True)
    rng = np.random.default_rng(len(sides))
    fs = [torch.from_numpy(W.uniform(2, n, seed=i)).cuda() for i, n in enumerate(sides)]
    u0 = [torch.from_numpy(rng.standard_normal((n, n))).cuda() for n in sides]
    b = B.BatchSolver(sides, precision=prec, **opts)
    for rows, its in ((0, 0), (5, 3)):
        for n in set(sides):
            b.set_tile_rows(n, rows)
            b.set_pass_iters(n, its)
        us = [u.clone() for u in u0]
        res = b.solve(fs, us, tol=1e-7, raise_on_status=False)  # one iteration a level need not converge
        for i, n in enumerate(sides):
            s = B.Solver(2, n, precision=prec, **opts)
            v = u0[i].clone()
            r = s.solve(fs[i], v, tol=1e-7, raise_on_status=False)
            assert res["cycles"][i] == r["cycles"] and res["statuses"][i] == r["status"], (n, i)
            assert np.array_equal(us[i].cpu().numpy(), v.cpu().numpy()), (n, i)
            assert res["relres"][i] == pytest.approx(r["final_relres"], rel=1e-13, abs=0)
            s.close()


def test_many_cycles(B, torch_cuda):
    """max_cycles past one launch of the one-workgroup problems, and
    problems that never reach the tolerance beside ones that do."""
    torch = torch_cuda
    sides = [17, 129, 33]
    fs = [torch.from_numpy(W.uniform(2, n, seed=n)).cuda() for n in sides]
    b = B.BatchSolver(sides, precision="fp64", max_cycles=70)
    us = [torch.zeros_like(f) for f in fs]
    res = b.solve(fs, us, tol=1e-300, raise_on_status=False)
    assert res["cycles"] == [70] * 3 and res["statuses"] == [7] * 3
    us = [torch.zeros_like(f) for f in fs]
    fs[1][5, 5] = float("nan")
    res = b.solve(fs, us, tol=1e-8, raise_on_status=False)
    assert res["statuses"] == [0, 6, 0] and res["cycles"][0] > 0
