"""Edges of the dense FP64 product's tiles: every configuration at column counts
around its 16-column chunks (whole pairs, an odd chunk, a partial one, none),
rows of odd leading dimension, several row tiles per workgroup, and the RBF map
from distance 0 down to kernel values that underflow."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from tests.helpers import assert_parity, dev, idx_dev

pytestmark = pytest.mark.gpu

RBF = (2, 0.7, 0.0, 1)
POLY = (1, 0.0, 1.0, 3)


@pytest.fixture(scope="module")
def K():
    from paper_2406_18001_amd import kdcd
    return kdcd


@pytest.mark.parametrize("n", [1, 4, 15, 16, 17, 31, 32, 33, 48, 50, 64, 79])
def test_every_config_at_chunk_edges(K, n):
    m, sb = 333, 70
    rng = np.random.default_rng(n)
    A = rng.standard_normal((m, n)) / np.sqrt(n)
    wide = torch.zeros(m, n + 3, dtype=torch.float64, device="cuda")   # odd rows start off 16-byte lines
    wide[:, :n] = dev(A)
    S = rng.integers(0, m, size=sb).astype(np.int32)
    beta = rng.standard_normal(m)
    try:
        for kk in (RBF, POLY):
            ok = O.Kernel(kk[0], sigma=kk[1], c=kk[2], degree=kk[3])
            r_ref, W_ref = O.kernel_rhs(A, ok, S, beta), O.kernel_block(A, ok, S, S)
            for cid in range(len(K.kdcd_tune_configs("f64"))):
                K.kdcd_tune_set("f64", n, sb, cid)
                for M in (dev(A), wide[:, :n]):
                    r, W = K.kdcd_kernel_rhs(M, kk, idx_dev(S), dev(beta), want_W=True)
                    assert_parity(r.cpu().numpy(), r_ref, 1e-11, f"r config {cid}")
                    assert_parity(W.cpu().numpy(), W_ref, 1e-12, f"W config {cid}")
    finally:
        K.kdcd_tune_set("f64", n, sb, -1)


@pytest.mark.parametrize("n", [24, 48])
def test_several_row_tiles_per_workgroup(K, n):
    """More row tiles than row groups (1024): ranges of one and two tiles."""
    m, sb = 64 * 1024 + 64 * 700 + 5, 20
    rng = np.random.default_rng(n)
    A = rng.standard_normal((m, n)) / np.sqrt(n)
    S = rng.integers(0, m, size=sb).astype(np.int32)
    beta = rng.standard_normal(m)
    ref = O.kernel_rhs(A, O.Kernel(O.RBF, sigma=0.7), S, beta)
    try:
        for cid in range(len(K.kdcd_tune_configs("f64"))):
            K.kdcd_tune_set("f64", n, sb, cid)
            r = K.kdcd_kernel_rhs(dev(A), RBF, idx_dev(S), dev(beta))
            assert_parity(r.cpu().numpy(), ref, 1e-11, f"config {cid}")
    finally:
        K.kdcd_tune_set("f64", n, sb, -1)


def test_rbf_values_over_their_range(K):
    """Distances from 0 to where exp underflows: each kernel value within 2 ulp of
    numpy's, subnormal values within one unit, zero below."""
    d = np.concatenate([[0.0], 2.0 ** np.arange(-60, 10.0), np.linspace(0.0, 780.0, 3000)])
    A = np.concatenate([[0.0], np.sqrt(d)]).reshape(-1, 1)
    m = A.shape[0]
    ref = np.exp(-(A[1:, 0] * A[1:, 0]))
    got = np.empty(m - 1)
    for j in range(0, m - 1, 500):        # W's first row: the sampled rows against row 0
        S = np.concatenate([[0], np.arange(1 + j, min(1 + j + 500, m))]).astype(np.int32)
        _, W = K.kdcd_kernel_rhs(dev(A), (2, 1.0, 0.0, 1), idx_dev(S), dev(np.zeros(m)), want_W=True)
        got[j:j + 500] = W.cpu().numpy()[0, 1:]
    normal = ref > 2.3e-308
    assert (np.abs(got - ref)[normal] <= 2 * np.spacing(ref[normal])).all()
    assert (np.abs(got - ref)[~normal] <= 2 * 5e-324).all()


@pytest.mark.parametrize("n,sb", [(33, 10), (48, 40), (17, 100)])
def test_every_batch_config(K, n, sb):
    m = 333
    rng = np.random.default_rng(sb)
    A = rng.standard_normal((m, n)) / np.sqrt(n)
    y = rng.standard_normal(m)
    lab = np.where(rng.standard_normal(m) > 0, 1.0, -1.0)
    idx = np.concatenate([rng.permutation(m)[:sb] for _ in range(3)]).astype(np.int32)
    specs = [("krr", 1e-3, 0.5, y), ("krr", 1e-2, 1.5, y), ("ksvm", 1.0, 0.5, lab)] * 7   # 21 problems
    refs = [O.bdcd_krr(A, yy, O.Kernel(O.RBF, sigma=sg), p, 1, 3 * sb, idx, s=sb)[0] if kind == "krr" else
            O.dcd_ksvm(A, yy, O.Kernel(O.RBF, sigma=sg), p, 3 * sb, idx, s=sb)[0]
            for kind, p, sg, yy in specs[:3]]
    cid16 = 16   # the batched FP64 table
    try:
        for cid in range(len(K.kdcd_tune_configs(cid16))):
            K.kdcd_tune_set(cid16, n, sb, cid)
            ps = [K.BatchProblem(kind, p, sg, dev(yy), torch.zeros(m, dtype=torch.float64, device="cuda"))
                  for kind, p, sg, yy in specs]
            K.kdcd_batch_solve(dev(A), K.Kernel(2, 1.0), 1, sb, 3 * sb, idx_dev(idx), ps)
            for i, q in enumerate(ps):
                assert_parity(q.alpha.cpu().numpy(), refs[i % 3], 1e-9, f"config {cid} problem {i}")
    finally:
        K.kdcd_tune_set(cid16, n, sb, -1)
