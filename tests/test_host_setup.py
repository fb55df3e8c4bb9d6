"""What operator setup asks of the HIP runtime."""
import ctypes

import numpy as np
import pytest

import host_library
from paper_1603_04334_amd import binding

pytestmark = pytest.mark.skipif(not host_library.available(), reason="needs hipcc")


def test_operator_setup_frees_nothing():
    """hipFree waits for the whole device: the server builds operators on its
    workers while others compute."""
    L = host_library.load()
    L.stub_reset()
    st, op = host_library.create(host_library.cluster((12, 11, 10), [((0, 3, 2), (5, 4, 7)), ((4, 0, 3), (6, 6, 6))]))
    assert st == 0
    assert not host_library.calls("hipFree", "hipFreeAsync")
    L.sparc_op_destroy(op)


def _waits_last(names, L, make):
    """make() -> (status, destroy); its last null-stream copy or fill is followed by a wait for that stream."""
    L.stub_reset()
    st, destroy = make()
    assert st == 0
    log = [c for c in host_library.calls() if c[0] in names or c[0] == "hipStreamSynchronize"]
    copies = [i for i, c in enumerate(log) if c[0] in names]
    waits = [i for i, c in enumerate(log) if c[0] == "hipStreamSynchronize" and c[1]["stream"] == 0]
    assert copies and waits and waits[-1] > copies[-1]
    destroy()


NULL_STREAM = ("hipMemcpy", "hipMemset")


def test_operator_setup_waits_for_its_copies():
    L = host_library.load()

    def make():
        st, op = host_library.create(host_library.cluster((12, 11, 10), [((0, 3, 2), (5, 4, 7))]))
        return st, lambda: L.sparc_op_destroy(op)

    _waits_last(NULL_STREAM, L, make)


@pytest.mark.parametrize("block", [(4, 4, 4), (2, 2, 2)])
def test_poisson_setup_waits_for_its_copies(block):
    L = host_library.load()

    def make():
        g = binding.sparc_grid()
        g.n[:] = [9, 10, 11]
        g.h, g.radius = 0.5, 6
        b = (ctypes.c_int32 * 3)(*block)
        h = ctypes.c_void_p()
        st = L.sparc_poisson_create(ctypes.byref(g), 6, ctypes.cast(b, ctypes.c_void_p), ctypes.byref(h))
        return st, lambda: L.sparc_poisson_destroy(h)

    _waits_last(NULL_STREAM, L, make)


@pytest.mark.parametrize("mode", [0, 1, 2, 3, 4, 5])
def test_batch_setup_waits_for_its_copies(mode):
    L = host_library.load()
    st, op = host_library.create(host_library.cluster((12, 12, 12), [((3, 3, 3), (5, 5, 5))]))
    assert st == 0
    X, Y = np.zeros((3, 1728)), np.zeros((3, 1728))

    def make():
        job = binding.sparc_batch_job(op, 0, X.ctypes.data, 1728, Y.ctypes.data, 1728, 3, 4, -1.0, 1.0, 2.0)
        h = ctypes.c_void_p()
        return L.sparc_batch_create(ctypes.byref(job), 1, mode, ctypes.byref(h)), lambda: L.sparc_batch_destroy(h)

    _waits_last(NULL_STREAM, L, make)
    L.sparc_op_destroy(op)


@pytest.mark.parametrize("ns,natoms,edge", [(1, 60, 12), (4, 8, 9), (70, 3, 7)])
@pytest.mark.parametrize("dtype", [binding.SPARC_F64, binding.SPARC_F32])
def test_admission_estimate_covers_a_cluster(ns, natoms, edge, dtype):
    """What the server reserves for a cluster against what its first request allocates."""
    L = host_library.load()
    rng = np.random.default_rng(3)
    n = 40
    cl = host_library.cluster((n, n, n), [(rng.integers(0, n - edge + 1, 3).tolist(), (edge,) * 3)
                                          for _ in range(natoms)], nproj=9)
    g, atoms, veff, keep = binding._cluster_arrays(cl)
    d = binding.sparc_cluster_desc(g, veff.ctypes.data_as(binding._dp), natoms, atoms, dtype, ns, 4, None, cl.nd, None, 1.0)
    L.stub_reset()
    st, op = host_library.create(cl)
    assert st == 0
    used = sum(c["bytes"] for _, c in host_library.calls("hipMalloc"))
    block = cl.nd * ns * (8 if dtype == binding.SPARC_F64 else 4)
    used += 2 * block + L.sparc_workspace_bytes(op, dtype, ns, 1) + L.sparc_rr_workspace_bytes(op, dtype, ns)
    used += 8 * ns * ns + L.sparc_rotate_workspace_bytes(dtype, ns) + L.sparc_lanczos_workspace_bytes(op, 40)
    reserved = L.sparc_cluster_footprint(ctypes.byref(d), 40)
    assert used <= reserved
    L.sparc_op_destroy(op)
