"""A solve that allocates its workspace is refused on a stream under capture; later calls
on other streams run as if it had not been made.  (The stream itself stays invalidated in
the runtime: it is the test's own and is destroyed.)"""
import ctypes

import pytest
import torch

from paper_2406_18001_amd import inputs
from tests.helpers import dev, idx_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [500, 40000])
@pytest.mark.parametrize("compute", ["f64", "bf16x3"])
def test_call_after_a_refused_one(m, compute):
    from paper_2406_18001_amd import kdcd as K
    hip = K._lib                                  # (looks symbols up in the runtime it links)
    d = inputs.dense_krr_c2(m=m, n=64, seed=1)
    A, y, idx = dev(d["A"]), dev(d["y"]), idx_dev(inputs.krr_indices(m, 4, 32, seed=0))
    ref = torch.zeros(m, dtype=torch.float64, device="cuda")
    K.kdcd_krr_solve(A, y, K.Kernel(2, 1.0), 1e-2, 4, 16, 32, idx, ref, compute=compute)
    K.kdcd_graph_cache_clear()                    # nothing kept: the next call allocates
    a = torch.zeros(m, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    st, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(st), 1) == 0
    assert hip.hipStreamBeginCapture(st, 1) == 0
    try:
        with pytest.raises(K.KdcdError):
            K.kdcd_krr_solve(A, y, K.Kernel(2, 1.0), 1e-2, 4, 16, 32, idx, a, compute=compute, stream=st.value)
    finally:
        assert hip.hipStreamEndCapture(st, ctypes.byref(graph)) != 0
        hip.hipStreamDestroy(st)
        hip.hipGetLastError()
    for stream in (torch.cuda.Stream(), None):
        a.zero_()
        torch.cuda.synchronize()
        K.kdcd_krr_solve(A, y, K.Kernel(2, 1.0), 1e-2, 4, 16, 32, idx, a, compute=compute, stream=stream)
        assert torch.equal(a, ref)
