"""Which kernels a CSR solve takes, without a GPU: the dense-panel product only where its
panel holds the sampled rows' columns and it is not the slower one."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PANEL, WAVE, HEAD, BROADCAST = "pp_product_kernel", "kblock_csr_wave_kernel", "kblock_csr_head_kernel", "kblock_csr_kernel"


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-fPIC", "-shared", os.path.join(HERE, "hip_stub.c"), "-o", so], check=True)
    return so


# rows of about avg entries, the longest of them, sampled rows, the caller's workspace?
@pytest.mark.parametrize("m,n,avg,longest,s,ws,kernel", [
    (30000, 500, 250, 370, 64, True, WAVE),           # the panel would overflow at every chunk
    (30000, 500, 250, 500, 64, True, WAVE),
    (30000, 500, 250, 370, 64, False, PANEL),
    (30000, 2000, 113, 170, 64, True, HEAD),
    (60000, 20000, 113, 170, 32, True, HEAD),         # a panel for eight rows
    (60000, 20000, 113, 9000, 32, True, HEAD),
    (60000, 20000, 113, 170, 48, False, PANEL),
    (20000, 2000, 113, 170, 24, False, HEAD),         # even rows, one dense-head chunk
    (20000, 2000, 113, 1700, 24, False, PANEL),
    (60000, 1000000, 113, 170, 1, False, BROADCAST),  # even rows, few sampled
    (60000, 1000000, 113, 900, 1, False, PANEL),
    (20000, 1000000, 1000, 1500, 1, True, WAVE),      # and code words in no cache
    (20000, 1000000, 1000, 1500, 4, True, PANEL),
    (20000, 20000, 1000, 1500, 1, False, PANEL),
    (19996, 1355191, 455, 16000, 64, True, PANEL),
    (30000, 50000, 50, 60, 32, False, HEAD),          # short rows
    (30000, 50000, 50, 60, 8, False, BROADCAST),
])
def test_kernel_of_a_solve(stub, m, n, avg, longest, s, ws, kernel):
    body = f"""
from tests.hip_host import *
put("row_max", {longest}, ctypes.c_uint64)
assert solve(csr({m}, {n}, {m * avg}), 1, {s}, {s} * 3, "svm", workspace={ws}) == 0
print(launched())
"""
    r = subprocess.run([sys.executable, "-c", body, stub], capture_output=True, text=True, timeout=120, cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stdout + r.stderr
    got = [k for k in (PANEL, WAVE, HEAD, BROADCAST) if k in r.stdout]
    # (a dense-head or panel chunk that may overflow has a gated kernel after it)
    assert got[0] == kernel
    assert r.stdout.count(kernel) >= 3
    # the panel memory is laid out for the kernel that reads it
    assert ("pp_init_kernel" in r.stdout) == (kernel == PANEL)


@pytest.mark.parametrize("longest,kernel,other", [(170, BROADCAST, PANEL), (900, PANEL, BROADCAST)])
@pytest.mark.parametrize("H", [5, 40])                # one graph of the whole call, a graph of a window
def test_kernel_of_a_graph(stub, longest, kernel, other, H):
    """The rows' lengths are looked at when the graph is captured; what runs around its
    replays is of the same kind, also when they have changed since."""
    body = f"""
from tests.hip_host import *
a = (f64 * 60000)()
A = csr(60000, 1000000, 60000 * 113)
for longest in ({longest}, 170, 900):
    put("row_max", longest, ctypes.c_uint64)
    assert solve(A, 1, 1, {H}, "svm", flags=GRAPH, alpha=a) == 0
print(launched())
"""
    r = subprocess.run([sys.executable, "-c", body, stub], capture_output=True, text=True, timeout=120, cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stdout + r.stderr
    # (a panel chunk that may overflow has a gated kernel of the other kind after it)
    assert kernel in r.stdout and (kernel == PANEL or other not in r.stdout)
    assert ("pp_init_kernel" in r.stdout) == (kernel == PANEL)
    assert r.stdout.count("csr_row_max_kernel") == 1
