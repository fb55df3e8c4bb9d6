"""Launch choices of the step kernels: what sparc_step_config reports can be
set again with sparc_op_set_launch."""
import ctypes

import pytest

import host_library
from paper_1603_04334_amd import binding

pytestmark = pytest.mark.skipif(not host_library.available(), reason="needs hipcc")


def _config(L, op, dtype, ns):
    v = [ctypes.c_int32() for _ in range(5)]
    assert L.sparc_step_config(op, dtype, ns, *[ctypes.byref(x) for x in v]) == 0
    return tuple(x.value for x in v)


@pytest.mark.parametrize("dtype", [binding.SPARC_F64, binding.SPARC_F32])
@pytest.mark.parametrize("n,ns", [((24, 24, 24), 8), ((40, 96, 96), 64), ((32, 160, 160), 60), ((30, 75, 92), 40),
                                  ((20, 46, 44), 220), ((16, 90, 164), 60), ((16, 61, 52), 300)])
@pytest.mark.parametrize("natoms", [0, 2])
def test_reported_config_can_be_set(n, ns, dtype, natoms):
    L = host_library.load()
    st, op = host_library.create(host_library.cluster(n, [((2, 2, 2), (3, 3, 3))] * natoms))
    assert st == 0
    config = _config(L, op, dtype, ns)
    assert L.sparc_op_set_launch(op, dtype, *config) == 0, (config, L.sparc_last_error())
    assert _config(L, op, dtype, ns) == config
    listed = config[:2] in [(32, 8), (32, 16), (32, 32), (32, 64), (64, 8), (64, 16), (64, 24), (64, 32), (80, 32),
                            (160, 24)]
    if not listed:  # a row-pair patch: one column per workgroup
        assert L.sparc_op_set_launch(op, dtype, *config[:4], 2) == binding.SPARC_E_ARG
    # and taken back
    assert L.sparc_op_set_launch(op, dtype, 0, 0, 0, 0, 0) == 0
    assert _config(L, op, dtype, ns) == config
    L.sparc_op_destroy(op)


def test_row_pair_patch_needs_a_whole_unit():
    L = host_library.load()
    st, op = host_library.create(host_library.cluster((40, 40, 3), []))
    assert st == 0
    assert L.sparc_op_set_launch(op, binding.SPARC_F32, 4, 40, 0, 0, 0) == binding.SPARC_E_ARG
    L.sparc_op_destroy(op)
