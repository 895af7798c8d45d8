"""The gradient of the learned relaxation where a workgroup takes several tiles:
its launch has at most 1024 workgroups, one per tile of 14 x 14 nodes up to a
lattice of side 450 and a second tile for some from there on (470: 1156 tiles;
513: 1369; 603: 1849, the last of each row one node short).

Tolerance, from what FP32 can give: the same formulas in plain FP32 torch are
off the FP64 oracle by some e; the kernels, also FP32 but summed in another
order and across workgroups in FP64, may be off by 4 e, and by eight roundings
(8 x 2^-23) of the largest gradient where e happens to be small."""
import numpy as np
import pytest

from oracle import learned as LO

pytestmark = pytest.mark.gpu


def plain_fp32(torch, x, r, a, hl, delta, w):
    """L and dL/dw in FP32 on the CPU, by torch's own differentiation."""
    import torch.nn.functional as F
    t = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32))
    x, r, delta, w = t(x), t(r), t(delta), t(w).requires_grad_(True)
    nm = x.shape[0]
    if a is None:
        face = [torch.ones(nm - 2, nm - 2)] * 4
    else:
        a = t(a)
        c = a[1:-1, 1:-1]
        face = [2.0 * c * q / (c + q) for q in (a[1:-1, :-2], a[1:-1, 2:], a[:-2, 1:-1], a[2:, 1:-1])]
    west, east, south, north = face

    def apply(v):
        c = v[1:-1, 1:-1]
        return (west * (c - v[1:-1, :-2]) + east * (c - v[1:-1, 2:]) + south * (c - v[:-2, 1:-1])
                + north * (c - v[2:, 1:-1]))

    rho = (np.float32(hl * hl) * r[1:-1, 1:-1] - apply(x)) / (((west + east) + south) + north)
    X = F.pad(torch.stack((rho, rho * (east - west) / (east + west), rho * (north - south) / (north + south))),
              (1, 1, 1, 1))
    mask = torch.zeros(nm, nm)
    mask[1:-1, 1:-1] = 1.0
    H = torch.relu(F.conv2d(X[None], w[:LO.NW1].view(LO.HID, 3, 3, 3), padding=1)) * mask
    z = delta - F.conv2d(H, w[LO.NW1:].view(1, LO.HID, 3, 3), padding=1)[0, 0] * mask
    inner = (slice(1, -1), slice(1, -1))
    loss = (z[inner] * apply(z)).sum() / (delta[inner] * apply(delta)).sum()
    loss.backward()
    return float(loss.detach()), w.grad.numpy().astype(np.float64)


@pytest.mark.parametrize("nm,var", [(9, True), (16, False), (17, True), (31, True), (64, True), (64, False), (129, True),
                                    (470, True), (470, False), (513, False), (603, True)])
def test_gradient(nm, var):
    import torch
    import paper_1108_2045_amd.homg as H
    print("gradient nm=%d var=%s" % (nm, var), flush=True)
    rng = np.random.default_rng(nm)
    f32 = lambda v: np.asarray(v, np.float32).astype(np.float64)
    mask = LO.interior_mask(nm)
    x, delta = f32(rng.standard_normal((nm, nm)) * mask), f32(rng.standard_normal((nm, nm)) * mask)
    r = f32(rng.standard_normal((nm, nm)) * (nm - 1) ** 2)
    a = f32(np.exp(rng.standard_normal((nm, nm)))) if var else None
    w = f32(LO.jacobi_weights(0.8) + 0.1 * rng.standard_normal(LO.NW))
    hl = 1.0 / (nm - 1)
    L, g = LO.loss_and_grad(x, r, a, hl, delta, w)
    L32, g32 = plain_fp32(torch, x, r, a, hl, delta, w)
    d = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).cuda() if v is not None else None
    got, _, loss = H.learn_grad(d(x), d(r), d(a), d(delta), d(w), hl)
    err, plain = np.max(np.abs(got.cpu().numpy() - g)), np.max(np.abs(g32 - g))
    big = np.max(np.abs(g))
    print("  off by %.2e of the largest gradient (plain FP32 %.2e); loss %.2e (%.2e)"
          % (err / big, plain / big, abs(loss / L - 1), abs(L32 / L - 1)), flush=True)
    assert err <= 4 * plain + 8 * 2.0 ** -23 * big
    assert abs(loss - L) <= 4 * abs(L32 - L) + 8 * 2.0 ** -23 * L
