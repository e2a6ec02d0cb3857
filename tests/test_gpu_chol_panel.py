"""The Cholesky panel of the Nystrom factor at the edges of its column groups and
panels, and its refusal of a matrix that is not positive definite."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from tests.helpers import assert_parity, dev, idx_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 2, 15, 16, 17, 33, 48, 49, 63, 64, 65, 80, 127, 129])
def test_factor_matches_oracle(r):
    from paper_2406_18001_amd import kdcd as K
    rng = np.random.default_rng(r)
    A = rng.standard_normal((200, 21)) / np.sqrt(21)
    L = rng.permutation(200)[:r].astype(np.int32)
    Phi = torch.empty(200, r, dtype=torch.float64, device="cuda")
    K.kdcd_nystrom_features(dev(A), K.Kernel(2, 1.0), idx_dev(L), 1e-4, Phi)
    ref = O.nystrom_features(A, O.Kernel(O.RBF, sigma=1.0), L, 1e-4)
    assert_parity(Phi.cpu().numpy(), ref, 1e-9, "Phi")


@pytest.mark.parametrize("pos", [0, 15, 16, 40, 63, 64, 90])
def test_not_positive_definite(pos):
    """Landmark `pos` is a row of zeros: its diagonal under the linear map is 0."""
    from paper_2406_18001_amd import kdcd as K
    A = np.eye(100, 110)
    A[pos] = 0.0
    with pytest.raises(K.KdcdError):
        K.kdcd_nystrom_features(dev(A), K.Kernel(0, 0.0), idx_dev(np.arange(100)), 0.0,
                                torch.empty(100, 100, dtype=torch.float64, device="cuda"))
