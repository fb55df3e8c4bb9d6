"""The nonlocal-force tables as the host builds them: every unit a lane may
read lies inside the table, also where an atom's cube spans a whole axis and
its arms along it are empty."""
import ctypes

import numpy as np
import pytest

import host_library

pytestmark = pytest.mark.skipif(not host_library.available(), reason="needs hipcc")

# one box: unit0, nunits, fun0, nf; an atom: three boxes, nproj, proj0
BOX = np.dtype([("unit0", "<i4"), ("nunits", "<i4"), ("fun0", "<i8"), ("nf", "<i4"), ("pad", "<i4")])
ATOM = np.dtype([("box", BOX, 3), ("nproj", "<i4"), ("proj0", "<i4")])


@pytest.mark.parametrize("n,ext", [((12, 12, 12), (5, 5, 5)), ((12, 5, 12), (5, 5, 5)), ((5, 12, 12), (5, 5, 5)),
                                   ((5, 5, 12), (5, 5, 5)), ((5, 5, 5), (5, 5, 5)), ((1, 1, 3), (1, 1, 3))])
def test_units_read_lie_in_the_table(n, ext):
    lo = [(n[d] - ext[d]) // 2 for d in range(3)]
    cl = host_library.cluster(n, [(lo, ext)] * 2)
    L = host_library.load()
    st, op = host_library.create(cl)
    assert st == 0
    L.stub_reset()
    ns = 3
    psi = np.zeros((ns, cl.nd))
    occ = np.ones(ns)
    force = np.zeros((2, 3))
    ws = np.zeros(max(1, L.sparc_force_workspace_bytes(op, ns)), dtype=np.uint8)
    st = L.sparc_nonlocal_force(op, 0, psi.ctypes.data, cl.nd, ns, occ.ctypes.data, force.ctypes.data, ws.ctypes.data,
                                ws.nbytes, None)
    assert st == 0
    size = {c["ptr"]: c["bytes"] for _, c in host_library.calls("hipMalloc")}
    up = [c for _, c in host_library.calls("hipMemcpy") if c["kind"] == 1]
    rec, units = up[0], up[1]
    assert rec["bytes"] == 2 * ATOM.itemsize and size[rec["dst"]] >= rec["bytes"]
    table = np.frombuffer(ctypes.string_at(rec["dst"], rec["bytes"]), dtype=ATOM)
    room = size[units["dst"]] // 8  # units of two integers
    assert sum(int(b["nunits"]) for a in table for b in a["box"]) <= room
    empty = 0
    for a in table:
        for b in a["box"]:
            # a lane past its share reads the box's first unit
            assert b["unit0"] + max(1, b["nunits"]) <= room
            empty += int(b["nunits"] == 0)
    assert (empty > 0) == (n[0] == ext[0] or n[1] == ext[1])
    L.sparc_op_destroy(op)
