"""What operator setup asks of the HIP runtime."""
import pytest

import host_library

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
