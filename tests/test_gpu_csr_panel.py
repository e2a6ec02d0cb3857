"""The dense-panel CSR product (rows of 112 and more stored entries on
average): every lanes-per-sampled-row width and its edges, rows shared by a
workgroup's waves, a panel too small for the chunk, infinities, determinism."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2406_18001_amd import inputs
from tests.helpers import assert_parity, dev, idx_dev
from tests.test_gpu_news20 import as_oracle, to_gpu

pytestmark = pytest.mark.gpu

RBF1 = (2, 1.0, 0.0, 1)
LINEAR = (0, 0.0, 0.0, 1)


@pytest.fixture(scope="module")
def K():
    from paper_2406_18001_amd import kdcd
    return kdcd


def make(lens, n, seed):
    rng = np.random.default_rng(seed)
    rows = [np.sort(rng.choice(n, L, replace=False)).astype(np.int32) for L in lens]
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    val = rng.standard_normal(int(row_ptr[-1])) / np.sqrt(max(1.0, float(np.mean(lens))))
    return {"row_ptr": row_ptr, "col_idx": np.concatenate(rows), "val": val, "m": len(lens), "n": n}


@pytest.fixture(scope="module")
def uneven():
    # empty rows, one entry, around the 64-entry step, the 256-entry batch and
    # the 2048 entries from which a workgroup shares the row
    rng = np.random.default_rng(3)
    lens = [0, 1, 63, 64, 65, 255, 256, 257, 511, 513, 2047, 2048, 2049, 2500, 2900, 0, 0]
    lens += list(rng.integers(0, 400, 113))
    c = make(lens, 3000, 5)
    c["val"][::97] = 0.0                      # stored zeros
    c["val"][::193] = -0.0
    return c


@pytest.mark.parametrize("kk", [LINEAR, RBF1])
@pytest.mark.parametrize("sb", [1, 8, 9, 16, 17, 32, 33, 64, 65, 130])
def test_panel_rhs(K, uneven, kk, sb):
    c = uneven
    assert c["row_ptr"][-1] >= 112 * c["m"]
    S = np.roll(np.arange(c["m"]), -10)[:sb].astype(np.int32)
    beta = np.random.default_rng(sb).standard_normal(c["m"])
    scale = np.sign(beta)
    ok = O.Kernel(kk[0], sigma=kk[1], c=kk[2], degree=kk[3])
    A = to_gpu(K, c)
    r, W = K.kdcd_kernel_rhs(A, kk, idx_dev(S), dev(beta), dev(scale), want_W=True)
    assert_parity(r.cpu().numpy(), O.kernel_rhs(as_oracle(c), ok, S, beta * scale), 1e-11, "r")
    assert_parity(W.cpu().numpy(), O.kernel_block(as_oracle(c), ok, S, S), 1e-12, "W")
    for _ in range(2):
        r1, W1 = K.kdcd_kernel_rhs(A, kk, idx_dev(S), dev(beta), dev(scale), want_W=True)
        assert torch.equal(r, r1) and torch.equal(W, W1)


@pytest.mark.parametrize("s", [4, 16, 70])
def test_panel_in_caller_workspace(K, uneven, s):
    """The smallest workspace holds a small panel: narrower chunks, and the
    broadcast kernel for chunks whose columns do not fit it."""
    c = uneven
    m, H = c["m"], 140
    y = np.where(np.arange(m) % 3 == 0, -1.0, 1.0)
    idx = inputs.ksvm_indices(m, H, seed=s)
    ref, _ = O.dcd_ksvm(as_oracle(c), y, O.Kernel(O.RBF, sigma=1.0), 1.0, H, idx, s=s)
    A = to_gpu(K, c)
    kern = K.Kernel(K.KERNEL_RBF, 1.0)
    ws = torch.empty(K.kdcd_workspace_bytes(0, A, kern, 1, s), dtype=torch.uint8, device="cuda")
    for w in (None, ws):
        alpha = torch.zeros(m, dtype=torch.float64, device="cuda")
        K.kdcd_ksvm_solve(A, dev(y), kern, 1.0, 1, s, H, idx_dev(idx), alpha, workspace=w)
        assert_parity(alpha.cpu().numpy(), ref, 1e-9, "alpha")


def test_panel_many_builds(K):
    """More builds than code words have epochs (4095), the epochs' reuse included."""
    c = make([150] * 20, 400, 9)
    y = np.where(np.arange(20) % 2 == 0, -1.0, 1.0)
    H = 4300
    idx = inputs.ksvm_indices(20, H, seed=1)
    ref, _ = O.dcd_ksvm(as_oracle(c), y, O.Kernel(0), 1.0, H, idx, s=1)
    alpha = torch.zeros(20, dtype=torch.float64, device="cuda")
    K.kdcd_ksvm_solve(to_gpu(K, c), dev(y), LINEAR, 1.0, 1, 1, H, idx_dev(idx), alpha)
    assert_parity(alpha.cpu().numpy(), ref, 1e-9, "alpha")


@pytest.mark.parametrize("sb", [4, 40])
def test_panel_infinite_value(K, sb):
    """An infinite stored value reaches only the sampled rows that store its column."""
    m, n = 60, 900
    c = make([130] * m, n, 11)
    e = int(c["row_ptr"][50]) + 17
    col = c["col_idx"][e]
    S = np.arange(sb, dtype=np.int32)
    stores = np.array([col in c["col_idx"][c["row_ptr"][j]:c["row_ptr"][j + 1]] for j in S])
    assert stores.any() and not stores.all()
    beta = np.random.default_rng(2).standard_normal(m)
    ref = O.kernel_rhs(as_oracle(c), O.Kernel(0), S, np.where(np.arange(m) == 50, 0.0, beta))
    row50 = O.kernel_block(as_oracle(c), O.Kernel(0), np.array([50], dtype=np.int32), S)[0]
    c["val"][e] = np.inf
    r = K.kdcd_kernel_rhs(to_gpu(K, c), LINEAR, idx_dev(S), dev(beta)).cpu().numpy()
    assert np.isinf(r[stores]).all()
    assert_parity(r[~stores], (ref + row50 * beta[50])[~stores], 1e-11, "r")
