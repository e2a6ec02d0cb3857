"""CSR solves on both sides of the dense-panel rule, against the oracle: the wave kernel
(long rows whose panel would overflow a caller's workspace; rows longer than its LDS panel),
the dense-head and broadcast kernels on even rows, the panel in the call's own memory."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2406_18001_amd import inputs
from tests.helpers import assert_parity, dev, idx_dev
from tests.test_gpu_csr_panel import make
from tests.test_gpu_news20 import as_oracle, to_gpu

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(4)
MATRICES = {
    "dense_even": make([250] * 90, 500, 1),
    "short_even": make([113] * 90, 1000, 2),
    "uneven": make([0, 1, 64, 65, 128, 129, 3072, 3073, 3500] + list(RNG.integers(0, 500, 70)), 4000, 3),
}


@pytest.mark.parametrize("name", MATRICES)
@pytest.mark.parametrize("s", [1, 7, 8, 9, 17, 24, 33, 70])
@pytest.mark.parametrize("kk", [(2, 1.0, 0.0, 1), (1, 0.0, 1.0, 3), (0, 0.0, 0.0, 1)])
def test_solves(name, s, kk):
    from paper_2406_18001_amd import kdcd as K
    c = MATRICES[name]
    m, H = c["m"], 3 * s + s // 2
    y = np.where(np.arange(m) % 3 == 0, -1.0, 1.0)
    idx = np.random.default_rng(s).integers(0, m, H).astype(np.int32)
    idx[0] = m - 1 if name != "uneven" else 8           # (the longest row among the first block's)
    ref, _ = O.dcd_ksvm(as_oracle(c), y, O.Kernel(kk[0], sigma=kk[1], c=kk[2], degree=kk[3]), 1.0, H, idx, s=s)
    A = to_gpu(K, c)
    ws = torch.empty(K.kdcd_workspace_bytes(0, A, K.Kernel(*kk), 1, s), dtype=torch.uint8, device="cuda")
    for kw in ({}, dict(workspace=ws), dict(flags=K.FLAG_GRAPH), dict(monitor_every=2)):
        a = torch.zeros(m, dtype=torch.float64, device="cuda")
        K.kdcd_ksvm_solve(A, dev(y), K.Kernel(*kk), 1.0, 1, s, H, idx_dev(idx), a, **kw)
        assert_parity(a.cpu().numpy(), ref, 1e-9, f"alpha {sorted(kw)}")


@pytest.mark.parametrize("name", MATRICES)
def test_krr_in_caller_workspace(name):
    from paper_2406_18001_amd import kdcd as K
    c = MATRICES[name]
    m, b, s, H = c["m"], 4, 6, 20
    y = np.random.default_rng(0).standard_normal(m)
    idx = inputs.krr_indices(m, b, H, seed=3)
    ref, _ = O.bdcd_krr(as_oracle(c), y, O.Kernel(O.RBF, sigma=1.0), 0.1, b, H, idx, s=s)
    A = to_gpu(K, c)
    ws = torch.empty(K.kdcd_workspace_bytes(1, A, K.Kernel(2, 1.0), b, s), dtype=torch.uint8, device="cuda")
    for kw in ({}, dict(workspace=ws)):
        a = torch.zeros(m, dtype=torch.float64, device="cuda")
        K.kdcd_krr_solve(A, dev(y), K.Kernel(2, 1.0), 0.1, b, s, H, idx_dev(idx), a, **kw)
        assert_parity(a.cpu().numpy(), ref, 1e-9, f"alpha {sorted(kw)}")
