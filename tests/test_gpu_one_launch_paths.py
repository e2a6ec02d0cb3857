"""That small dense K-SVM solves do run in one launch, and what follows when that launch
gives up (its wait set to end at once): the ordinary launches from the alpha of the call."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2406_18001_amd import inputs
from tests.helpers import dev, idx_dev

pytestmark = pytest.mark.gpu


@pytest.fixture
def K():
    from paper_2406_18001_amd import kdcd
    kdcd._lib.kdcd_one_launch_count.restype = ctypes.c_int64
    yield kdcd
    kdcd._lib.kdcd_one_launch_polls(-1)


def counts(K):
    return np.array([K._lib.kdcd_one_launch_count(0), K._lib.kdcd_one_launch_count(1)])


def problem(K, m, n, s, outer=37):
    rng = np.random.default_rng(m + n + s)
    A = dev(rng.standard_normal((m, n)) / np.sqrt(n))
    y = dev(np.where(rng.standard_normal(m) > 0, 1.0, -1.0))
    H = outer * s - (s > 1)
    idx = idx_dev(inputs.ksvm_indices(m, H, seed=s))
    alpha0 = dev(rng.random(m) * 0.5)

    def solve(**kw):
        a, tr = alpha0.clone(), torch.full((H,), 7.0, dtype=torch.float64, device="cuda")
        K.kdcd_ksvm_solve(A, y, K.Kernel(2, 0.05), 0.8, 1, s, H, idx, a, trace=tr, **kw)
        return a, tr
    ws = torch.empty(K.kdcd_workspace_bytes(0, A, K.Kernel(2, 0.05), 1, s), dtype=torch.uint8, device="cuda")
    return solve, ws


# (the sizes of test_gpu_svm_one_launch.py, whose comparisons say nothing if the path is not taken)
SIZES = [(1, 3, 1), (63, 16, 1), (64, 17, 2), (65, 64, 7), (640, 65, 16), (700, 255, 17), (2001, 256, 3), (1990, 64, 32),
         (4100, 31, 1), (12000, 48, 8), (2000, 256, 1), (1500, 50, 8)]


@pytest.mark.parametrize("m,n,s", SIZES)
def test_path_is_taken(K, m, n, s):
    solve, ws = problem(K, m, n, s)
    before = counts(K)
    solve()
    assert (counts(K) - before == [1, 0]).all()
    solve(workspace=ws)
    assert (counts(K) - before == [1, 0]).all()


@pytest.mark.parametrize("m,n,s", [(1, 3, 1), (65, 64, 7), (700, 255, 17), (2001, 256, 3), (12000, 48, 8)])
@pytest.mark.parametrize("polls", [0, 1, 3])
def test_giving_up(K, m, n, s, polls):
    """polls 0: in the first block.  1, 3: some block, or none."""
    solve, ws = problem(K, m, n, s)
    ref = solve(workspace=ws)
    before = counts(K)
    K._lib.kdcd_one_launch_polls(polls)
    for _ in range(5):
        got = solve()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    ended, gave_up = counts(K) - before
    assert ended + gave_up == 5 and (polls > 0 or gave_up == 5)
    K._lib.kdcd_one_launch_polls(-1)
    got = solve()
    assert torch.equal(got[0], ref[0]) and (counts(K) - before == [ended + 1, gave_up]).all()
