"""A C++ exception out of a library call (rocBLAS, rocSOLVER or the HIP runtime)
fails the request it happens in, with the exception's text, and nothing else:
the process, the other requests and the server go on."""
import ctypes
import os
import subprocess
import sys
import time

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path[:0] = [os.path.dirname(HERE), HERE]

import numpy as np  # noqa: E402

import host_library  # noqa: E402
from paper_1603_04334_amd import binding  # noqa: E402

pytestmark = pytest.mark.skipif(not host_library.available(), reason="needs hipcc")

FILL = ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t)


@FILL
def _fill(dst, src, nbytes):
    """What the host reads back: ascending values (coefficients, Ritz values),
    zero where a solver leaves its status (one integer, or behind the values)."""
    n = nbytes // 8
    v = 1.0 + 0.5 * np.arange(n)
    if n not in (0, 40, 39):
        v[-1] = 0.0
    ctypes.memset(dst, 0, nbytes)
    ctypes.memmove(dst, v.ctypes.data, 8 * n)


def _child(where, anywhere=False):
    L = host_library.load()
    L.stub_d2h(_fill)
    cfg = binding.sparc_server_cfg(0, 2, 40, 0, 0.0)
    srv = ctypes.c_void_p()
    assert L.sparc_server_create(ctypes.byref(cfg), ctypes.byref(srv)) == 0
    keep = []

    def submit(cid, ns, release=0):
        cl = host_library.cluster((12, 12, 12), [((3, 3, 3), (5, 5, 5))])
        g, atoms, veff, k = binding._cluster_arrays(cl)
        X0, v0 = np.zeros((ns, cl.nd)), np.ones(cl.nd)
        d = binding.sparc_cluster_desc(g, veff.ctypes.data_as(binding._dp), 1, atoms, 0, ns, 4, X0.ctypes.data, cl.nd,
                                       v0.ctypes.data, float(ns))
        keep.append((k, atoms, X0, v0, d))
        job = binding.sparc_filter_job(cid, ctypes.pointer(d), release, None)
        t = ctypes.c_uint64()
        assert L.sparc_filter_submit(srv, ctypes.byref(job), ctypes.byref(t)) == 0
        return t.value

    def wait(t):
        r = binding.sparc_job_result()
        end = time.time() + 60
        while L.sparc_filter_poll(srv, t, ctypes.byref(r)) == binding.SPARC_PENDING:
            assert time.time() < end
            time.sleep(0.001)
        return r

    if anywhere:
        # the call throws from here until the request and its clean-up are done
        L.stub_throw(where.encode())
        srv = ctypes.c_void_p()
        assert L.sparc_server_create(ctypes.byref(cfg), ctypes.byref(srv)) == 0
        for cid, release in ((1, 0), (2, 1)):
            r = wait(submit(cid, 70, release))
            print(where, r.status, r.error.decode(), flush=True)
        assert L.sparc_server_destroy(srv) == 0
        L.stub_throw(b"")
        srv = ctypes.c_void_p()
        assert L.sparc_server_create(ctypes.byref(cfg), ctypes.byref(srv)) == 0
        ok = wait(submit(3, 70, release=1))
        assert ok.status == 0, ok.error
        assert L.sparc_server_destroy(srv) == 0
        print("child ok", flush=True)
        return
    used = ctypes.c_uint64()
    for cid in (1, 2):
        L.stub_throw(where.encode())
        r = wait(submit(cid, 70))
        assert r.status == binding.SPARC_E_HIP and b"wrong index for variant" in r.error, (r.status, r.error)
        L.stub_throw(b"")
    # the failed clusters gave their memory back; later requests run
    ok = wait(submit(3, 70, release=1))
    assert ok.status == 0, ok.error
    assert L.sparc_server_stats(srv, None, None, None, ctypes.byref(used)) == 0 and used.value == 0
    log = host_library.calls("hipMallocAsync", "hipFreeAsync")
    assert ({c["ptr"] for n, c in log if n == "hipMallocAsync" and c["ptr"]}
            == {c["ptr"] for n, c in log if n == "hipFreeAsync" and c["ptr"]})
    if where.startswith("roc"):
        # a handle a call was thrown out of is not used again
        assert len(host_library.calls("rocblas_create_handle")) == 3
    assert L.sparc_server_destroy(srv) == 0
    print("child ok", flush=True)


@pytest.mark.parametrize("where", ["rocsolver_dpotrf", "rocblas_dtrsm", "rocsolver_dsyevd", "hipMallocAsync"])
def test_exception_fails_its_request_only(where):
    host_library.load()
    r = subprocess.run([sys.executable, os.path.abspath(__file__), where], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("where", [
    "hipSetDevice", "hipStreamCreateWithFlags", "hipStreamSynchronize", "hipFreeAsync", "hipFree", "hipStreamDestroy",
    "hipEventRecord", "hipEventQuery", "roctxRangePushA", "roctxRangePop", "rocblas_create_handle",
    "rocblas_set_stream"])
def test_exception_outside_a_request_leaves_the_process(where):
    """The worker's own calls, the clean-up after a request and what destructors
    call: none of them ends the process, and a later server runs its requests."""
    host_library.load()
    r = subprocess.run([sys.executable, os.path.abspath(__file__), where, "anywhere"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stdout + r.stderr


def test_exception_in_a_direct_call_is_a_status():
    """sparc_rayleigh_ritz and the GEMM of sparc_rotate called directly."""
    code = """
import ctypes, numpy as np, host_library
from paper_1603_04334_amd import binding
L = host_library.load()
st, op = host_library.create(host_library.cluster((12, 12, 12), []))
nd, ns = 1728, 70
Y, theta, evec = np.zeros((ns, nd)), np.zeros(ns), np.zeros((ns, ns))
ws = np.zeros(L.sparc_rr_workspace_bytes(op, 0, ns), dtype=np.uint8)
for name in (b"rocsolver_dpotrf", b"rocblas_dtrsm", b"rocsolver_dsyevd"):
    L.stub_throw(name)
    st = L.sparc_rayleigh_ritz(op, 0, Y.ctypes.data, nd, ns, theta.ctypes.data_as(binding._dp), evec.ctypes.data,
                               ws.ctypes.data, ws.nbytes, None)
    assert st == binding.SPARC_E_HIP and b"wrong index for variant" in L.sparc_last_error(), L.sparc_last_error()
ns = 300
Y, out, Q = np.zeros((ns, nd)), np.zeros((ns, nd)), np.zeros((ns, ns))
ws = np.zeros(L.sparc_rotate_workspace_bytes(0, ns), dtype=np.uint8)
L.stub_throw(b"rocblas_dgemm")
st = L.sparc_rotate(0, Y.ctypes.data, nd, nd, ns, Q.ctypes.data, out.ctypes.data, nd, ws.ctypes.data, ws.nbytes, None)
assert st == binding.SPARC_E_HIP and b"wrong index for variant" in L.sparc_last_error(), L.sparc_last_error()
print("child ok")
"""
    host_library.load()
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([os.path.dirname(HERE), HERE]))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stdout + r.stderr


if __name__ == "__main__":
    _child(sys.argv[1], len(sys.argv) > 2)
