"""The training kernels' matrix-core contractions against the FP64 oracle at
lattice sides around their tiles (14 owned nodes, 16 of a row per instruction)
and for weights that are no BF16 values.

Tolerance: every FP32 sum has at most 27 + 16 + 196 terms in a row, so its
rounding error is below 239 eps = 2.9e-5 of the sum of magnitudes; a gradient's
magnitudes exceed its largest value by at most 10 on these inputs."""
import numpy as np
import pytest

from oracle import learned as LO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


@pytest.mark.parametrize("var", [False, True])
@pytest.mark.parametrize("nm", [3, 4, 15, 16, 17, 18, 30, 31, 45, 230])
def test_gradient_and_forward(torch_cuda, nm, var):
    torch = torch_cuda
    import paper_1108_2045_amd.homg as H
    print("train contractions nm=%d var=%s" % (nm, var), flush=True)
    rng = np.random.default_rng(nm)
    f32 = lambda v: np.asarray(v, np.float32)
    mask = LO.interior_mask(nm)
    x, delta = f32(rng.standard_normal((nm, nm)) * mask), f32(rng.standard_normal((nm, nm)) * mask)
    r = f32(rng.standard_normal((nm, nm)) * (nm - 1) ** 2)
    a = f32(np.exp(rng.standard_normal((nm, nm)))) if var else None
    w = f32(LO.jacobi_weights(0.8) + 0.1 * rng.standard_normal(LO.NW))
    hl = 1.0 / (nm - 1)
    d = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda() if v is not None else None
    L, g = LO.loss_and_grad(x.astype(np.float64), r.astype(np.float64), None if a is None else a.astype(np.float64), hl,
                            delta.astype(np.float64), w.astype(np.float64))
    got, _, loss = H.learn_grad(d(x), d(r), d(a), d(delta), d(w), hl)
    assert loss == pytest.approx(L, rel=3e-4)
    assert np.max(np.abs(got.cpu().numpy() - g)) <= 3e-4 * np.max(np.abs(g))
    y = torch.zeros((nm, nm), dtype=torch.float32, device="cuda")
    H.learn_forward(d(x), d(r), d(a), d(w), hl, y)
    X = LO.features(x.astype(np.float64), r.astype(np.float64), None if a is None else a.astype(np.float64), hl)
    _, _, want = LO.forward(X, w.astype(np.float64))
    assert np.max(np.abs(y.cpu().numpy() - want)) <= 3e-5 * 10 * np.max(np.abs(want))
