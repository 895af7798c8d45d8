"""What the batched solver prepares on the host: its cost and its memory."""
import time

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


def test_making_a_batch_is_linear_in_its_problems(B, torch_cuda):
    """16000 problems of side 129 against 2000: eight times the work.  A walk
    over all problems for each of them would make it 64 times; the line at 20
    with 0.05 s for what does not depend on the count lies between."""
    def seconds(count):
        best = 1e9
        for _ in range(2):
            torch_cuda.cuda.synchronize()
            t = time.perf_counter()
            b = B.BatchSolver([129] * count, precision="bf16")
            best = min(best, time.perf_counter() - t)
            b.close()
        print("batch of %d made in %.4f s" % (count, best), flush=True)
        return best
    seconds(10)
    few = seconds(2000)
    assert seconds(16000) <= 20 * few + 0.05


def held(torch, make):
    """(device memory the handle made by make() holds, the handle)"""
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    h = make()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0], h


def test_lists_do_not_grow_with_the_iterations(B, torch_cuda):
    """A level of many iterations repeats one launch: its lists are kept once
    (a list per launch was 190 MB here, 20 GB at the largest side)."""
    small, h = held(torch_cuda, lambda: B.BatchSolver([8193], precision="bf16", max_i=8))
    h.close()
    many, h = held(torch_cuda, lambda: B.BatchSolver([8193], precision="bf16", max_i=8192))
    h.close()
    print("8193^2: %d MB with 8 iterations a level, %d MB with 8192" % (small >> 20, many >> 20), flush=True)
    assert many <= small + (64 << 20)


@pytest.mark.parametrize("sides,prec,max_i,its", [([257, 129, 513, 129], "fp64", 40, {129: 3}),
                                                  ([1025, 129], "bf16", 21, {1025: 2}),
                                                  ([2049, 513, 129], "fp32", 13, {2049: 1, 513: 4})])
def test_many_iterations_equal_single_solves(B, torch_cuda, sides, prec, max_i, its):
    """Levels of many passes, of different numbers in each problem: bit for bit
    as single solves."""
    torch = torch_cuda
    print("batch lists %s %s max_i=%d %s" % (sides, prec, max_i, its), flush=True)
    fs = [torch.from_numpy(W.uniform(2, n, seed=i)).cuda() for i, n in enumerate(sides)]
    us = [torch.zeros_like(f) for f in fs]
    b = B.BatchSolver(sides, precision=prec, max_i=max_i, max_cycles=3)
    for n, k in its.items():
        b.set_pass_iters(n, k)
    res = b.solve(fs, us, tol=1e-300, raise_on_status=False)
    for i, n in enumerate(sides):
        s = B.Solver(2, n, precision=prec, max_i=max_i)
        v = torch.zeros_like(fs[i])
        s.solve_cycles(fs[i], v, 3)
        assert res["cycles"][i] == 3 and np.array_equal(us[i].cpu().numpy(), v.cpu().numpy()), (n, i)
        s.close()


def test_settings_take_no_memory_in_a_solve(B, torch_cuda):
    """Tile rows and pass iterations changed between solves: nothing is
    allocated (level 0's iterates were, and the lists), on a stream of the
    caller's, and the results stay."""
    torch = torch_cuda
    sides = [513] * 8 + [129, 33]
    fs = [torch.from_numpy(W.uniform(2, n, seed=i)).cuda() for i, n in enumerate(sides)]
    b = B.BatchSolver(sides, precision="fp64")
    us = [torch.zeros_like(f) for f in fs]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):  # (a stream's first use takes memory of the runtime's own)
        first = b.solve(fs, us, tol=1e-8)
        want = [u.cpu().numpy() for u in us]
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for rows, its in ((1, 1), (64, 2), (5, 3), (0, 0)):
        for n in set(sides):
            b.set_tile_rows(n, rows)
            b.set_pass_iters(n, its)
        with torch.cuda.stream(s):
            for u in us:
                u.zero_()
            res = b.solve(fs, us, tol=1e-8)
            got = [u.cpu().numpy() for u in us]
        print("rows %d, iterations %d: %d bytes less" % (rows, its, free - torch.cuda.mem_get_info()[0]), flush=True)
        assert torch.cuda.mem_get_info()[0] >= free
        assert res["cycles"] == first["cycles"]
        assert all(np.array_equal(u, v) for u, v in zip(got, want))


def tuned(B, torch, sides, path=None):
    """seconds a tuning run takes"""
    fs = [torch.from_numpy(W.uniform(2, n, seed=i % 3)).cuda() for i, n in enumerate(sides)]
    us = [torch.zeros_like(f) for f in fs]
    b = B.BatchSolver(sides, precision="fp32")
    b.solve(fs, us, tol=1e-2)
    for u in us:
        u.zero_()
    t = time.perf_counter()
    b.tune(fs, us, tol=1e-2, cache_path=path)
    return time.perf_counter() - t


def test_tuner_leaves_out_sides_without_stages(B, torch_cuda):
    """Problems of side up to 65 read neither setting: the tuner times no
    candidates for them (4 solves against 28 for as many problems of side 129)."""
    small, staged = tuned(B, torch_cuda, [65] * 200), tuned(B, torch_cuda, [129] * 200)
    print("tuned in %.4f s (side 65), %.4f s (side 129)" % (small, staged), flush=True)
    assert small <= 0.5 * staged


def test_tuner_cache_is_kept_per_kind_of_batch(B, torch_cuda, tmp_path):
    """What was chosen for a batch whose passes run on tiles is not taken for
    one of the same sides whose passes walk, nor the other way round; each is
    found again for its own."""
    path = tmp_path / "tiles.txt"
    lines = []
    for sides in ([129, 257, 33], [129, 257, 33] * 40, [257, 33, 129], [129, 257, 33] * 41):
        tuned(B, torch_cuda, sides, str(path))
        lines.append([ln.split() for ln in path.read_text().split("\n") if ln.strip()])
    assert [len(v) for v in lines] == [3, 6, 6, 6]
    assert len({ln[0] for ln in lines[-1]}) == 2
