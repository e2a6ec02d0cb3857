"""K-SVM solves with up to 16 sampled rows sum the product's partials in the
recurrence: the same bits as a profiled solve, which keeps the finish pass, at the
edges of s, of the row groups and of their batches."""
import numpy as np
import pytest
import torch

from paper_2406_18001_amd import inputs
from tests.helpers import dev, idx_dev
from tests.test_gpu_csr_panel import make
from tests.test_gpu_news20 import to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [1, 2, 15, 16, 17])
@pytest.mark.parametrize("m", [1, 15, 500, 512 * 16, 512 * 16 + 1, 40000])
@pytest.mark.parametrize("csr", [True, False])
def test_same_bits_as_with_the_finish_pass(s, m, csr):
    from paper_2406_18001_amd import kdcd as K
    rng = np.random.default_rng(m + s)
    if csr:
        A = to_gpu(K, make(rng.integers(1, 12, m), 400, seed=m))
    else:
        A = dev(rng.standard_normal((m, 300)) / 17)        # too wide for the one-launch solve
    y = dev(np.where(rng.standard_normal(m) > 0, 1.0, -1.0))
    H = 5 * s + s // 2
    idx = idx_dev(inputs.ksvm_indices(m, H, seed=s))
    out = []
    for profile in (False, True):
        a = torch.zeros(m, dtype=torch.float64, device="cuda")
        tr = torch.full((H,), 7.0, dtype=torch.float64, device="cuda")
        K.kdcd_ksvm_solve(A, y, K.Kernel(2, 0.3), 1.0, 1, s, H, idx, a, trace=tr, profile=profile)
        out.append((a, tr))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert float(out[0][0].abs().sum()) > 0
