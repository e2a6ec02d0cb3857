"""Host code of the kept workspaces, without a GPU: what is kept is idle memory that any
later call may use."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """Runs a body of Python in a child process over the stub runtime."""
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-fPIC", "-shared", os.path.join(HERE, "hip_stub.c"), "-o", so], check=True)

    def run(body):
        r = subprocess.run([sys.executable, "-c", "from tests.hip_host import *\n" + body, so], capture_output=True,
                           text=True, timeout=120, cwd=os.path.dirname(HERE))
        assert r.returncode == 0, r.stdout + r.stderr
    return run


def test_kept_for_the_next_call(host):
    host("""
A = dense(3000, 40)
assert solve(A, 4, 16, 64) == 0 and get("mallocs") == 1
assert solve(A, 4, 16, 64) == 0 and get("mallocs") == 1
lib.kdcd_graph_cache_clear()
assert get("held", size) == 0
""")


@pytest.mark.parametrize("call", ["solve(A, 4, 16, 64)", "solve(A, 4, 16, 64, compute=BF16X3)",
                                  "lib.kdcd_sampler_select(ctypes.addressof(keys), 3000, 16, f64(0.5), ctypes.c_uint64(1), i64(0), ctypes.addressof(out), None)"])
def test_memory_of_a_capture_is_not_kept(host, call):
    """A call on a stream under capture fails, and the memory that it was given belongs to
    that graph: the next call takes its own."""
    host(f"""
A = dense(3000, 40)
keys, out = (ctypes.c_float * 3000)(), (i32 * 16)()
lib.kdcd_sampler_select.argtypes = [P, i64, i32, f64, ctypes.c_uint64, i64, P, P]
put("capturing", 1)
assert {call} != 0 and get("captured_mallocs") == 1
put("capturing", 0)
assert {call} == 0 and get("mallocs") == 1 and get("uses_captured") == 0
""")


def test_memory_of_a_failed_wait_is_not_kept(host):
    """The stream could not be waited for: its work may still run."""
    host("""
A = dense(3000, 40)
put("sync_error", 999)
assert solve(A, 4, 16, 64) == -7 and get("mallocs") == 1
put("sync_error", 0)
assert solve(A, 4, 16, 64) == 0 and get("mallocs") == 2
""")


# calls whose own workspace holds more than they need: Grams ahead, the full CSR panel
# (graphs too), the exchange words of the one-launch solve
CALLS = {
    "gram": ("A = dense(3000, 64)", "solve(A, 8, 64, 64 * 20, compute=BF16X3, flags=F, alpha=a)", "1, *W(A), 8, 64, BF16X3"),
    "panel": ("A = csr(2000, 100000, 400000)", "solve(A, 1, 64, 64 * 20, 'svm', flags=F, alpha=a)", "0, *W(A), 1, 64, F64"),
    "one_launch": ("A = dense(7000, 64)", "solve(A, 1, 32, 32 * 20, 'svm', flags=F, alpha=a)", "0, *W(A), 1, 32, F64"),
}
SETUP = """
a = (f64 * 200000)()
W = lambda A: (ctypes.byref(A), ctypes.byref(RBF))
F = %d
%s
need = lib.kdcd_workspace_bytes(%s)
"""


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("name", CALLS)
def test_least_memory_will_do(host, name, graph):
    A, call, ws = CALLS[name]
    host(SETUP % (graph, A, ws) + f"""
put("memory", need + (64 << 10), size)          # (64 KiB: a graph's window of indices)
assert {call} == 0 and {call} == 0
assert get("largest", size) <= need + (64 << 10)
put("memory", 1 << 40, size)
stub.stub_forget()
assert {call} == 0                              # and with the memory, all of it
assert get("largest", size) >= need + (80 << 10) or {graph and name == "one_launch"}
""")


def test_least_memory_of_a_product(host):
    host("""
A = csr(2000, 100000, 400000)
need = lib.kdcd_workspace_bytes(0, ctypes.byref(A), ctypes.byref(RBF), 1, 64, F64)
put("memory", need + 4096, size)
r = (f64 * 64)()
assert lib.kdcd_kernel_rhs(ctypes.byref(A), ctypes.byref(RBF), 4096, 64, 4096, None, r, None, F64, None) == 0
""")


@pytest.mark.parametrize("call", ["solve(B, 4, 16, 16 * 40, flags=GRAPH)", "lib.kdcd_sampler_create(ctypes.byref(P()), ctypes.c_uint64(1))"])
def test_kept_memory_makes_way(host, call):
    """Memory that is only kept does not fail an allocation."""
    host(f"""
A, B = dense(2000000, 40), dense(3000, 40)
assert solve(A, 4, 16, 64) == 0
put("memory", get("held", size) + 4096, size)
assert {call} == 0
""")
