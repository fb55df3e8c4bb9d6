"""Launch shapes of the Lanczos steps."""
import ctypes

import numpy as np
import pytest

import host_library
from paper_1603_04334_amd import binding

pytestmark = pytest.mark.skipif(not host_library.available(), reason="needs hipcc")


def test_lds_does_not_grow_with_the_step_count():
    """1 <= k <= N_d is accepted: no launch may ask for LDS per step (8 bytes
    a step would pass a workgroup's 64 KB at k = 8192)."""
    L = host_library.load()
    st, op = host_library.create(host_library.cluster((12, 12, 12), [((3, 3, 3), (5, 5, 5))]))
    assert st == 0
    most = {}
    for k in (20, 1500):
        v0, theta = np.ones(1728), np.zeros(k)
        ws = np.zeros(L.sparc_lanczos_workspace_bytes(op, k), dtype=np.uint8)
        L.stub_reset()
        # (the stand-in's coefficients are zero: a breakdown after the launches)
        st = L.sparc_lanczos(op, k, v0.ctypes.data, None, None, theta.ctypes.data_as(binding._dp), ws.ctypes.data,
                             ws.nbytes, None)
        assert st == binding.SPARC_E_BREAKDOWN
        launches = [c for _, c in host_library.calls("hipLaunchKernel")]
        assert len(launches) > 3 * k
        most[k] = max(c["lds"] for c in launches)
    assert most[1500] == most[20]
    L.sparc_op_destroy(op)
