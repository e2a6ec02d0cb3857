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
