"""CSR K-SVM solves build the next block's dense-head panel beside the recurrence:
the same bits as solves of one block each, which build their own panels, at the
edges of the chunks, with shorter last blocks, chunks too large for the panel, by
graph windows; and the oracle's iterate."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from tests.helpers import assert_parity, dev, idx_dev
from tests.test_gpu_csr_panel import make
from tests.test_gpu_news20 import as_oracle, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [17, 32, 33, 64, 65])
@pytest.mark.parametrize("blocks,last", [(2, 0), (5, 1), (4, 16), (21, 17)])
@pytest.mark.parametrize("long_rows", [False, True])
def test_same_bits_as_single_blocks(s, blocks, last, long_rows):
    from paper_2406_18001_amd import kdcd as K
    rng = np.random.default_rng(s + blocks)
    lens = rng.integers(0, 60, 900)
    if long_rows:
        lens[:90] = 250                               # 32 of these exceed the panel's 4096 entries
    c = make(lens, 3000, seed=s)
    m, H = c["m"], blocks * s + last
    A, y = to_gpu(K, c), np.where(rng.standard_normal(m) > 0, 1.0, -1.0)
    idx = rng.integers(0, 100 if long_rows else m, H).astype(np.int32)
    kern = K.Kernel(1, 0.0, 1.0, 3)
    whole = torch.zeros(m, dtype=torch.float64, device="cuda")
    K.kdcd_ksvm_solve(A, dev(y), kern, 0.7, 1, s, H, idx_dev(idx), whole)
    graph = torch.zeros_like(whole)
    K.kdcd_ksvm_solve(A, dev(y), kern, 0.7, 1, s, H, idx_dev(idx), graph, flags=K.FLAG_GRAPH)
    single = torch.zeros_like(whole)
    for k in range(0, H, s):
        n = min(s, H - k)
        K.kdcd_ksvm_solve(A, dev(y), kern, 0.7, 1, n, n, idx_dev(idx[k:k + n]), single)
    assert torch.equal(whole, single) and torch.equal(whole, graph)
    ref, _ = O.dcd_ksvm(as_oracle(c), y, O.Kernel(O.POLY, c=1.0, degree=3), 0.7, H, idx, s=s)
    assert_parity(whole.cpu().numpy(), ref, 1e-9, "alpha")
