"""Host code of the one-launch K-SVM solve, without a GPU: which solves take it, and what
they do when its launch is refused or gives up."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-fPIC", "-shared", os.path.join(HERE, "hip_stub.c"), "-o", so], check=True)

    def run(body):
        r = subprocess.run([sys.executable, "-c", "from tests.hip_host import *\n" + body, so], capture_output=True,
                           text=True, timeout=120, cwd=os.path.dirname(HERE))
        assert r.returncode == 0, r.stdout + r.stderr
    return run


@pytest.mark.parametrize("tile", [0, 3, 5])
def test_tuned_on_a_tall_matrix(host, tile):
    """A tile that the autotuner has found for n and s on a tall matrix."""
    host(f"""
lib.kdcd_tune_set.argtypes = [i32, i64, i32, i32]
for sb in (8, 4):
    assert lib.kdcd_tune_set(0, 64, sb, {tile}) == 0
assert solve(dense(2000, 64), 1, 8, 8 * 20 + 4, "svm") == 0
assert get("coop_launches") == 1 and "kblock_f64" not in launched()
""")


def test_refused_launch(host):
    host("""
put("coop_refused", 1)
assert solve(dense(2000, 64), 1, 8, 160, "svm") == 0
assert get("coop_launches") == 0 and launched().count("ksvm_recur_kernel") == 20
""")


def test_launch_that_gives_up(host):
    """Alpha is what it was when the ordinary launches take over."""
    host("""
put("coop_gives_up", 1)
alpha = (f64 * 2000)(*[0.25 + 1e-3 * i for i in range(2000)])
before = list(alpha)
assert solve(dense(2000, 64), 1, 8, 160, "svm", alpha=alpha) == 0
assert get("coop_launches") == 1 and launched().count("ksvm_recur_kernel") == 20
assert list(alpha) == before                      # (no kernel has run)
""")


@pytest.mark.parametrize("what", ["workspace=True", "flags=GRAPH"])
def test_not_taken(host, what):
    host(f"""
assert solve(dense(2000, 64), 1, 8, 160, "svm", {what}) == 0
assert get("coop_launches") == 0
""")
