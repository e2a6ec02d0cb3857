"""Freed workspaces are kept for later calls: solves of
several sizes from several threads and streams give what they give alone, and
kdcd_graph_cache_clear returns the memory."""
import threading

import pytest
import torch

from paper_2406_18001_amd import inputs
from tests.helpers import dev, idx_dev

pytestmark = pytest.mark.gpu


def solve(K, m, stream=None):
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    A = torch.randn(m, 64, generator=g, dtype=torch.float64, device="cuda") / 8
    y = torch.sin(A[:, 0])
    idx = idx_dev(inputs.krr_indices(m, 4, 3 * 16, seed=m))
    a = torch.zeros(m, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for _ in range(4):
        a.zero_()
        torch.cuda.synchronize()
        K.kdcd_krr_solve(A, y, K.Kernel(2, 1.0), 0.1, 4, 16, 3 * 16, idx, a, compute="bf16x3", stream=stream)
    torch.cuda.synchronize()
    return a.cpu()


def test_threads_and_streams():
    from paper_2406_18001_amd import kdcd as K
    sizes = [300, 5000, 70000, 300000]              # workspaces from under 1 MB to 80 MB and more
    alone = [solve(K, m) for m in sizes]
    got = [None] * len(sizes)

    def run(i):
        got[i] = solve(K, sizes[i], torch.cuda.Stream())

    ts = [threading.Thread(target=run, args=(i,)) for i in range(len(sizes))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert all(torch.equal(x, z) for x, z in zip(alone, got))


def test_memory_is_given_back():
    from paper_2406_18001_amd import kdcd as K
    solve(K, 1500000)
    torch.cuda.empty_cache()
    held = torch.cuda.mem_get_info()[0]
    K.kdcd_graph_cache_clear()
    free = torch.cuda.mem_get_info()[0]
    assert free >= held + (300 << 20)               # most of the two 16-bit copies' 384 MB
