"""What the batched solver prepares on the host: its cost and its memory."""
import time

import pytest

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
