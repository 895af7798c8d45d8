"""Every entry point on a stream of the caller's that the null stream does not
wait for, with its inputs still being written there by work enqueued before:
bit for bit as on the default stream."""
import numpy as np
import pytest

import workloads as W
from oracle import learned as LO

pytestmark = pytest.mark.gpu


def calls(P, torch):
    """{name: call on the current stream, inputs given by a function that makes
    them there}"""
    def solve(d, n, prec, make, var=False, learned=False, **opts):
        s = P.Solver(d, n, precision=prec, stencil=P.DIFFUSION_5PT_2D if var else None, **opts)

        def call():
            a, f = make((n,) * d)
            u = torch.zeros_like(f)
            if var:
                s.set_coefficient(a)
            if learned:
                w = torch.from_numpy(LO.jacobi_weights(0.7).astype(np.float32)).cuda(non_blocking=False)
                s.set_smoother(P.LEARNED, w)
            r = s.solve(f, u, tol=1e-8)
            return [u, torch.tensor(r["history"])]
        return call

    def residual(make):
        s = P.Solver(2, 257)

        def call():
            a, f = make((257, 257))
            r = torch.zeros_like(f)
            return [torch.tensor(s.residual(f, a, r)), r]
        return call

    def batch(make):
        sides = [17, 65, 129, 257]
        b = P.BatchSolver(sides, precision="fp32")

        def call():
            b.set_pass_iters(257, 2)  # the lists are made again, and go up on this stream
            fs = [make((n, n))[1] for n in sides]
            us = [torch.zeros_like(f) for f in fs]
            b.solve(fs, us, tol=1e-8)
            return us
        return call

    def train(make):
        w = torch.from_numpy(LO.jacobi_weights(0.7).astype(np.float32)).cuda()

        def call():
            a, f = make((129, 129))
            x = (0.1 * f).float()
            g, e, loss = P.homg.learn_grad(x, (f * 1e4).float(), a.float(), (f + 0.01).float(), w, 1.0 / 128)
            return [g.clone(), torch.tensor([e, loss])]
        return call

    return {
        "small": lambda m: solve(2, 33, "fp64", m), "2d": lambda m: solve(2, 257, "fp32", m),
        "3d": lambda m: solve(3, 33, "bf16", m), "3d small": lambda m: solve(3, 17, "fp64", m),
        "diffusion": lambda m: solve(2, 129, "fp64", m, var=True),
        "learned": lambda m: solve(2, 129, "fp64", m, var=True, learned=True),
        "pow2": lambda m: solve(2, 512, "fp64", m, grid_layout="pow2"),
        "in cycle": lambda m: solve(2, 129, "fp64", m, restriction="in_cycle"),
        "residual": residual, "batch": batch, "train": train,
    }


@pytest.mark.parametrize("name", ["small", "2d", "3d", "3d small", "diffusion", "learned", "pow2", "in cycle",
                                  "residual", "batch", "train"])
def test_own_stream(name):
    import torch
    import paper_1108_2045_amd as P
    import paper_1108_2045_amd.homg  # noqa: F401
    print("own stream: %s" % name, flush=True)
    busy = torch.randn(4096, 4096, device="cuda") / 64.0
    host = {}

    def make(shape):
        """(a, f), written late: after some milliseconds of products"""
        if shape not in host:
            rng = np.random.default_rng(shape[0])
            f = W.uniform(len(shape), shape[0], seed=1)
            host[shape] = [torch.from_numpy(np.exp(0.5 * rng.standard_normal(shape))).cuda(), torch.from_numpy(f).cuda()]
            torch.cuda.synchronize()
        t = busy
        for _ in range(8):
            t = t @ busy
        late = (t[0, 0] * 0.0).double()
        return [v + late for v in host[shape]]

    call = calls(P, torch)[name](make)
    want = [v.cpu().numpy() for v in call()]
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    for _ in range(2):
        with torch.cuda.stream(s):
            out = call()
            got = [v.cpu().numpy() for v in out]
        assert all(np.array_equal(g, v) for g, v in zip(got, want)) and len(got) == len(want)
