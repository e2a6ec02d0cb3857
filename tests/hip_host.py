"""For a child process: libkdcd.so over tests/hip_stub.c (host memory, kernels logged and
not run), so that the library's host code runs without a GPU.  sys.argv[1] is the built stub."""
import ctypes
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before the library: its symbols win
lib = ctypes.CDLL(os.environ.get("KDCD_LIBRARY") or os.path.join(ROOT, "paper_2406_18001_amd", "libkdcd.so"))
i32, i64, f64, P, size = ctypes.c_int32, ctypes.c_int64, ctypes.c_double, ctypes.c_void_p, ctypes.c_size_t
F64, BF16X3, GRAPH = 0, 4, 1


class Matrix(ctypes.Structure):
    _fields_ = [("format", i32), ("reserved", i32), ("m", i64), ("n", i64), ("ld", i64), ("nnz", i64), ("values", P),
                ("row_ptr", P), ("col_idx", P)]


class Kernel(ctypes.Structure):
    _fields_ = [("kind", i32), ("degree", i32), ("sigma", f64), ("c", f64)]


class Options(ctypes.Structure):
    _fields_ = [("compute", i32), ("loss", i32), ("snapshot_every", i32), ("flags", i32), ("snapshots", P), ("trace", P),
                ("workspace", P), ("workspace_bytes", size), ("profile", P), ("monitor_every", i32), ("reserved", i32),
                ("tol", f64), ("outer_done", P), ("rel_err", P), ("monitor_log", P), ("monitor_log_len", i64)]


lib.kdcd_workspace_bytes.restype = size
lib.kdcd_workspace_bytes.argtypes = [i32, P, P, i32, i32, i32]
for _f in (lib.kdcd_ksvm_solve, lib.kdcd_krr_solve):
    _f.argtypes = [P, P, P, f64, i32, i32, i64, P, P, P, P]
lib.kdcd_kernel_rhs.argtypes = [P, P, P, i32, P, P, P, P, i32, P]
stub.stub_launched.restype = ctypes.c_char_p


def get(name, t=ctypes.c_int):
    return t.in_dll(stub, "stub_" + name).value


def put(name, value, t=ctypes.c_int):
    t.in_dll(stub, "stub_" + name).value = value


def launched():
    return stub.stub_launched().decode()


def dense(m, n):
    return Matrix(0, 0, m, n, n, 0, 4096, None, None)         # (A is never read here)


def csr(m, n, nnz):
    return Matrix(1, 0, m, n, n, nnz, 4096, 4096, 4096)


RBF = Kernel(2, 1, 1.0, 0.0)
LIVE = []


def solve(A, b, s, H, problem="krr", compute=F64, workspace=False, flags=0, alpha=None):
    """The status of a solve; workspace: of kdcd_workspace_bytes, by the caller."""
    o = Options()
    o.compute, o.loss, o.flags = compute, 1, flags
    if workspace:
        need = lib.kdcd_workspace_bytes(1 if problem == "krr" else 0, ctypes.byref(A), ctypes.byref(RBF), b, s, compute)
        buf = ctypes.create_string_buffer(need + 256)
        LIVE.append(buf)
        o.workspace, o.workspace_bytes = -(-ctypes.addressof(buf) // 256) * 256, need
    if alpha is None:
        alpha = (f64 * A.m)()
    LIVE.append(alpha)
    f = lib.kdcd_krr_solve if problem == "krr" else lib.kdcd_ksvm_solve
    return f(ctypes.byref(A), 4096, ctypes.byref(RBF), 1.0, b, s, H, 4096, ctypes.addressof(alpha), ctypes.byref(o), None)
