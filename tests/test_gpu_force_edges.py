"""Edges of the nonlocal-force launches against the oracle: workgroups that take
all nodes of an atom and 32 orbitals (from 1024 of them), launches split into 4
or 16 parts of the nodes (16 below 32 atom-and-orbital blocks), 1 to 4 tiles of
functions, orbital counts beside the 16- and 32-column blocks, cubes and arms
cut by the walls or reaching over the whole axis, grids below one 4-node unit.

Both sides sum in FP64 and differ by rounding order only: the bound is 1e-10 of
the largest force component, as in test_gpu_force.py."""
import numpy as np
import pytest

import oracle
from paper_1603_04334_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-10


def _run(cl, ns, dtype, seed, small_ws=False):
    from paper_1603_04334_amd import binding as b
    rng = np.random.default_rng(seed)
    X = torch.from_numpy(rng.standard_normal((ns, cl.nd))).to(dtype).cuda()
    occ = rng.uniform(0.0, 1.0, ns)
    g = torch.from_numpy(occ).cuda()
    op = b.Operator(cl)
    ws = torch.empty(4 * 4 * cl.nproj_total * ns * 8, dtype=torch.uint8, device="cuda") if small_ws else None
    f = op.nonlocal_force(X, g, ws=ws)
    torch.cuda.synchronize()
    got = f.cpu().numpy()
    ref = oracle.nonlocal_force(cl, X.double().cpu().numpy(), occ)
    err = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"force {cl.n} natoms {len(cl.atoms)} ns {ns} {dtype} small_ws {small_ws}: rel err {err:.2e}", flush=True)
    assert err <= TOL
    return got


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nproj", [1, 4, 7, 9, 13, 16])
@pytest.mark.parametrize("ns", [1, 15, 17, 33])
def test_tiles_of_functions_and_orbitals(nproj, ns, dtype):
    """1 to 4 tiles of functions (the second atom has one projector less, at
    least 1); 16 parts, and 4 in the smallest workspace."""
    cl = inputs.make_cluster((17, 22, 19), 0.45, 2, 6, 2, seed=nproj, min_dist=1.0, margin=1.0)
    rng = np.random.default_rng(nproj)
    for a, p in zip(cl.atoms, (nproj, max(1, nproj - 1))):
        a.chi = np.concatenate([a.chi, a.chi * rng.uniform(0.5, 1.5, a.chi.shape)])[:p].copy()
        a.gamma = rng.uniform(-2.0, 2.0, p)
    _run(cl, ns, dtype, ns)
    _run(cl, ns, dtype, ns, small_ws=True)


@pytest.mark.parametrize("natoms,ns", [(16, 17), (32, 40), (63, 520), (64, 512), (65, 481)])
def test_whole_and_split_launches(natoms, ns):
    """32 blocks (4 parts) and both sides of 1024 whole workgroups."""
    cl = inputs.make_cluster((43, 38, 45), 0.5, natoms, 6, 1, seed=natoms, min_dist=0.0)
    _run(cl, ns, torch.float32, natoms)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [(1, 1, 3), (3, 1, 1), (2, 3, 5), (1, 9, 2), (12, 1, 7)])
def test_tiny_grids(n, dtype):
    """Rows and grids shorter than a unit, arms cut on both sides or absent."""
    cl = inputs.make_cluster(n, 0.6, 1, 6, 1, seed=3, min_dist=0.0, margin=0.0)
    _run(cl, 6, dtype, 5)
