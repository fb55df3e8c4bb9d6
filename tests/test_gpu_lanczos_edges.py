"""Edges of the Lanczos step against the oracle: rows of whole and cut 16-byte
units, a single node per row (the scalar step), grids below one patch, no
atoms, more projectors than the fused update keeps (the separate scatter),
small and large start vectors.

Short runs, before any Ritz value converges: the coefficients then differ by
the rounding of FP64 sums over N_d terms amplified over k steps, below 1e-10 of
the spectrum here; the bound is 1e-9."""
import numpy as np
import pytest

import oracle
from paper_1603_04334_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(cl, k, scale=1.0):
    from paper_1603_04334_amd import binding
    v0 = inputs.lanczos_start(cl.nd, 3)
    alpha, beta, theta = binding.Operator(cl).lanczos(k, torch.from_numpy(scale * v0).cuda())
    ra, rb, rt = oracle.lanczos(cl, k, v0)
    top = np.abs(rt).max()
    err = max(np.abs(alpha - ra).max(), np.abs(np.asarray(beta)[: k - 1] - rb).max(), np.abs(theta - rt).max()) / top
    print(f"lanczos {cl.n} atoms {len(cl.atoms)} k {k}: rel err {err:.2e}", flush=True)
    assert err <= 1e-9


@pytest.mark.parametrize("n", [(9, 7, 12), (9, 7, 13), (3, 11, 1), (1, 1, 40), (2, 5, 3), (33, 17, 34), (18, 31, 33)])
def test_grids_without_atoms(n):
    _check(inputs.free_cluster(n, 0.5), 6)


@pytest.mark.parametrize("n", [(20, 18, 24), (20, 18, 25), (17, 19, 33), (16, 40, 1)])
@pytest.mark.parametrize("lmax", [0, 2])
def test_grids_with_atoms(n, lmax):
    _check(inputs.make_cluster(n, 0.5, 2, 6, lmax, seed=5, min_dist=0.0, margin=0.0), 8)


@pytest.mark.parametrize("natoms", [227, 228])
def test_projector_table_limit(natoms):
    """2043 and 2052 projectors: both sides of the table of the fused update."""
    _check(inputs.make_cluster((64, 60, 62), 0.5, natoms, 6, 2, seed=9, min_dist=0.0), 5)


@pytest.mark.parametrize("scale", [1e-100, 1e100])
def test_start_vector_scale(scale):
    _check(inputs.make_cluster((20, 18, 25), 0.5, 2, 6, 1, seed=5, min_dist=0.0), 8, scale)
