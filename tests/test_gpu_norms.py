"""The residual's walks and norms at every side: short 3D walks, the sum of
f^2 taken in the first residual pass, and the history stored in host memory.

Tolerances: each residual is a sum of at most 8 FP64 terms, so it lies within
16 eps of sum |terms|; the norms are sums of squares (relative 1e-12 covers
n^d eps / 2 with pairwise partial sums)."""
import numpy as np
import pytest

import workloads as W
from oracle import homg as O

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


@pytest.mark.parametrize("d,n", [(2, 3), (2, 5), (2, 65), (2, 257), (3, 3), (3, 5), (3, 9), (3, 17), (3, 33),
                                 (3, 65), (3, 129)])
def test_residual_and_norms(B, torch_cuda, d, n):
    torch = torch_cuda
    print("residual d=%d n=%d" % (d, n), flush=True)
    rng = np.random.default_rng(900 + n)
    f = W.uniform(d, n, seed=n)
    u = rng.standard_normal((n,) * d)  # Dirichlet data on the boundary too
    s = B.Solver(d, n)
    fd, ud = torch.from_numpy(f).cuda(), torch.from_numpy(u).cuda()
    r = torch.zeros_like(fd)
    rel = s.residual(fd, ud, r)
    ro, so = O.residual(d, n, f, u)
    scale = 4 * d * np.max(np.abs(u)) * (n - 1.0) ** 2 + np.max(np.abs(f))
    inner = (slice(1, -1),) * d
    assert np.max(np.abs(r.cpu().numpy() - ro)[inner]) <= 16 * 2.3e-16 * scale
    want = np.sqrt(so) / np.sqrt(O.norm2_interior(d, n, f))
    assert rel == pytest.approx(want, rel=1e-12)
    # a solve's history holds the same norms, whatever its batches of cycles
    res = s.solve_cycles(fd, ud, 0)
    assert res["history"] == [res["relres0"]] and res["relres0"] == pytest.approx(want, rel=1e-12)
    res = s.solve_cycles(fd, ud, 5)
    assert len(res["history"]) == 6 and res["history"][0] == pytest.approx(want, rel=1e-12)
    floor = 16 * 2.3e-16 * 4 * d * (n - 1.0) ** 2 * np.linalg.norm(ud.cpu().numpy()) / np.linalg.norm(f[inner])
    assert res["final_relres"] == pytest.approx(s.residual(fd, ud), rel=1e-9, abs=floor)
