"""Grams formed ahead in the low-precision lookahead loop, whose ring of buffers wraps
after 16 blocks: the same bits as with one buffer (a caller's workspace), for fewer
blocks than the ring has, one more, several rounds and a partial last block."""
import numpy as np
import pytest
import torch

from paper_2406_18001_amd import inputs
from tests.helpers import dev, idx_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s", [(1, 256), (1, 257), (3, 87), (8, 32), (8, 64)])
@pytest.mark.parametrize("blocks", [2, 16, 17, 18, 19, 35])
@pytest.mark.parametrize("compute", ["bf16x3", "bf16", "f32"])
def test_same_bits_as_one_buffer(b, s, blocks, compute):
    from paper_2406_18001_amd import kdcd as K
    m, n = 600 + b, 45
    rng = np.random.default_rng(blocks)
    A = dev(rng.standard_normal((m, n)) / np.sqrt(n))
    y = dev(rng.standard_normal(m))
    kern = K.Kernel(2, 1.0)
    ws = torch.empty(K.kdcd_workspace_bytes(1, A, kern, b, s, compute=compute), dtype=torch.uint8, device="cuda")
    for H in (blocks * s, blocks * s - s // 2):
        idx = idx_dev(inputs.krr_indices(m, b, H, seed=s))
        out = []
        for kw in (dict(workspace=ws), {}, dict(profile=True), dict(flags=K.FLAG_GRAPH)):
            a = torch.full((m,), 0.1, dtype=torch.float64, device="cuda")
            tr = torch.full((H * b,), 7.0, dtype=torch.float64, device="cuda")
            kw["flags"] = kw.get("flags", 0) | K.FLAG_LOOKAHEAD
            info = K.kdcd_krr_solve(A, y, kern, 1e-2, b, s, H, idx, a, compute=compute, trace=tr, **kw)
            if kw.get("profile"):
                # the recurrences run in the products' launches, but for the last block's
                assert info["recur_launches"] == 1
            out.append((a, tr))
        for a, tr in out[1:]:
            assert torch.equal(a, out[0][0]) and torch.equal(tr, out[0][1])
