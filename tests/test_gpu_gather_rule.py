"""Both sides of the line between projections gathered in the step's tail and by
a workgroup per atom and 16 columns: a column's result does not depend on how
many columns are applied with it, bit for bit."""
import pytest

import oracle
from paper_1603_04334_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,natoms", [((32, 32, 32), 64), ((26, 31, 29), 70)])  # whole units, cut rows
def test_columns_alone_and_with_more(n, natoms):
    from paper_1603_04334_amd import binding
    cl = inputs.make_cluster(n, 0.5, natoms, 6, 1, seed=3, min_dist=0.0, margin=2.0)
    op = binding.Operator(cl)
    X = inputs.device_orbitals(cl.nd, 257, 4, torch.float32).contiguous()
    line = -(-1024 // natoms) * 16  # columns from which the pairs reach 1024
    few, many = line - 16, line + 1
    assert many <= 257
    a, b = op.h_apply(X[:few]), op.h_apply(X[:many])
    assert torch.equal(a, b[:few])
    bounds = (-3.0, 1.5, oracle.upper_bound(cl))
    a, b = op.cheb_filter(X[:few], 4, *bounds), op.cheb_filter(X[:many], 4, *bounds)
    assert torch.equal(a, b[:few])
