"""How many iterations a Poisson solve enqueues before it looks whether it is done."""
import ctypes

import numpy as np
import pytest

import host_library
from paper_1603_04334_amd import binding

pytestmark = pytest.mark.skipif(not host_library.available(), reason="needs hipcc")


@pytest.mark.parametrize("guess,max_iter,first", [(0, 100, 24), (1, 100, 12), (1, 5, 5), (0, 7, 7), (0, 0, 0)])
def test_iterations_before_the_first_read(guess, max_iter, first):
    """A solve from a guess may need a few iterations only: it reads its flag after twelve."""
    L = host_library.load()
    g = binding.sparc_grid()
    g.n[:] = [12, 13, 14]
    g.h, g.radius = 0.5, 6
    b = (ctypes.c_int32 * 3)(4, 4, 4)
    h = ctypes.c_void_p()
    assert L.sparc_poisson_create(ctypes.byref(g), 6, ctypes.cast(b, ctypes.c_void_p), ctypes.byref(h)) == 0
    n = 12 * 13 * 14
    charge, phi = np.zeros(n), np.zeros(n)
    ws = np.zeros(L.sparc_poisson_workspace_bytes(h), dtype=np.uint8)
    L.stub_reset()

    @ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t)
    def fill(dst, src, nbytes):  # never converged
        ctypes.memset(dst, 0, nbytes)
        ctypes.memmove(dst, np.array([0x7fffffff], dtype=np.int32).ctypes.data, 4)

    L.stub_d2h(fill)
    try:
        st = L.sparc_poisson_solve(h, charge.ctypes.data, phi.ctypes.data, guess, 1e-8, max_iter, None, None, None,
                                   ws.ctypes.data, ws.nbytes, None)
    finally:
        L.stub_d2h(None)
    assert st == 0
    runs, count = [], 0
    for name, c in host_library.calls("hipLaunchKernel", "hipStreamSynchronize"):
        if name == "hipStreamSynchronize":
            runs.append(count)
        elif "xp_update_kernel" in c["name"]:
            count += 1
    assert count == max_iter
    assert runs[0] == 0 and (runs[1] if len(runs) > 1 else 0) == first
    assert max(np.diff(runs), default=0) <= 24
    L.sparc_poisson_destroy(h)
