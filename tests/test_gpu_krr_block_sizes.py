"""K-RR with the block sizes that have their own recurrence variant and no other
parity test: partial last blocks, repeated coordinates, the longest blocks."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_18001_amd import inputs
from tests.helpers import assert_parity, dev, idx_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [3, 5, 6, 7, 9])
@pytest.mark.parametrize("s", [1, 2, 13, 0])            # 0: as long as a block can be
def test_iterate_matches_oracle(b, s):
    from paper_2406_18001_amd import kdcd as K
    s = s or 512 // b
    m, H = 4 * b * min(s, 20) // 3 + 40, 3 * s + s // 2       # blocks share many coordinates
    rng = np.random.default_rng(10 * b + s)
    A = rng.standard_normal((m, 19)) / 4
    y, alpha0 = rng.standard_normal(m), rng.standard_normal(m)
    idx = inputs.krr_indices(m, b, H, seed=s)
    a, tr = dev(alpha0), dev(np.full(H * b, 7.0))
    K.kdcd_krr_solve(dev(A), dev(y), K.Kernel(2, 0.7), 0.1, b, s, H, idx_dev(idx), a, trace=tr)
    ref, ref_tr = O.bdcd_krr(A, y, O.Kernel(O.RBF, sigma=0.7), 0.1, b, H, idx, alpha0=alpha0, s=s)
    assert_parity(a.cpu().numpy(), ref, 1e-9, "alpha")
    assert_parity(tr.cpu().numpy(), ref_tr, 1e-9, "trace")
