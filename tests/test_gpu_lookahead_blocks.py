"""The lookahead recurrence at the edges of its element pairs and waves: odd and
even s*b, every b it takes, last blocks of other lengths, many repeated
coordinates; against the oracle and the loop without lookahead."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_18001_amd import inputs
from tests.helpers import assert_parity, dev, idx_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s", [(1, 256), (1, 257), (1, 385), (1, 511), (2, 129), (3, 87), (3, 170), (4, 65), (5, 77),
                                 (6, 64), (7, 55), (7, 73), (8, 32), (8, 33), (8, 63), (8, 64)])
@pytest.mark.parametrize("compute", ["f64", "f32", "bf16x3"])
def test_matches_oracle(b, s, compute):
    from paper_2406_18001_amd import kdcd as K
    m, n, H = 600 + s, 32, 3 * s + s // 3
    rng = np.random.default_rng(100 * b + s)
    A = rng.standard_normal((m, n)) / np.sqrt(n)
    y, alpha0 = rng.standard_normal(m), 0.1 * rng.standard_normal(m)
    idx = inputs.krr_indices(m, b, H, seed=s)
    out = {}
    for flags in (K.FLAG_LOOKAHEAD, K.FLAG_SERIAL):
        a, tr = dev(alpha0), dev(np.full(H * b, 7.0))
        K.kdcd_krr_solve(dev(A), dev(y), K.Kernel(2, 0.7), 0.1, b, s, H, idx_dev(idx), a, trace=tr, compute=compute,
                         flags=flags)
        out[flags] = a.cpu().numpy(), tr.cpu().numpy()
    if compute == "f64":
        ref = O.bdcd_krr(A, y, O.Kernel(O.RBF, sigma=0.7), 0.1, b, H, idx, alpha0=alpha0, s=s)
    else:
        ref = out[K.FLAG_SERIAL]     # the same low-precision r up to the order of its FP64 sums, and FP64 kernel rows
    tol = 1e-9 if compute == "f64" else 1e-5
    assert_parity(out[K.FLAG_LOOKAHEAD][0], ref[0], tol, "alpha")
    assert_parity(out[K.FLAG_LOOKAHEAD][1], ref[1], tol, "trace")
