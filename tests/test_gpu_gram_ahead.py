"""Low-precision solves form the FP64 Grams of several index blocks in one launch
when the call has the memory: the same bits as block by block (which a caller's
workspace selects), for fewer blocks than one launch takes, one more, several
launches and a partial last block, with and without the lookahead loop."""
import numpy as np
import pytest
import torch

from paper_2406_18001_amd import inputs
from tests.helpers import dev, idx_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("problem,b,s", [("krr", 1, 16), ("krr", 8, 64), ("krr", 3, 7), ("krr", 4, 1),
                                         ("ksvm", 1, 64), ("ksvm", 1, 5)])
@pytest.mark.parametrize("H", [2, 17, 18, 35])              # index blocks, the last one partial
@pytest.mark.parametrize("mode", ["plain", "graph", "monitor"])
def test_same_bits_as_block_by_block(problem, b, s, H, mode):
    from paper_2406_18001_amd import kdcd as K
    m, n = 1500 + b, 45
    rng = np.random.default_rng(H)
    A = dev(rng.standard_normal((m, n)) / np.sqrt(n))
    y = dev(np.where(rng.standard_normal(m) > 0, 1.0, -1.0))
    H = H * s - s // 2
    idx = idx_dev(inputs.krr_indices(m, b, H, seed=s))
    kern = K.Kernel(2, 1.0)
    solve, reg, pid = ((K.kdcd_krr_solve, 1e-2, 1) if problem == "krr" else (K.kdcd_ksvm_solve, 1.0, 0))
    out = []
    own = dict(flags=K.FLAG_GRAPH) if mode == "graph" else dict(monitor_every=4) if mode == "monitor" else {}
    ws = torch.empty(K.kdcd_workspace_bytes(pid, A, kern, b, s, compute="bf16x3"), dtype=torch.uint8, device="cuda")
    for kw in (dict(workspace=ws), own):
        a = torch.full((m,), 0.1, dtype=torch.float64, device="cuda")
        tr = torch.full((H * b,), 7.0, dtype=torch.float64, device="cuda")
        solve(A, y, kern, reg, b, s, H, idx, a, compute="bf16x3", trace=tr, **kw)
        out.append((a, tr))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
