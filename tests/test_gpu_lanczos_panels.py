"""Lanczos runs longer than one panel of re-orthogonalisation coefficients
(1024), on a grid small enough for its whole spectrum.

T_k is the projection of H on the Krylov space, so its eigenvalues interlace
those of H: lambda_j <= theta_j <= lambda_{n-k+j} for every j.  A basis that
loses orthogonality (a panel left out, or taken twice) shows copies of
converged eigenvalues, which break the left side at once.  Semi-orthogonality
(below sqrt(eps)) keeps T_k the projection up to O(n eps |H|), 3e-13 here; the
bound is 1e-11."""
import numpy as np
import pytest

import oracle
from paper_1603_04334_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1024, 1025, 1026, 1200])
def test_interlacing(k):
    from paper_1603_04334_amd import binding
    cl = inputs.make_cluster((11, 12, 10), 0.5, 2, 6, 1, seed=5, min_dist=0.0, margin=0.0)
    rng = np.random.default_rng(2)
    cl.veff = cl.veff + rng.standard_normal(cl.nd)  # no symmetry: the eigenvalues are distinct
    lam = np.linalg.eigvalsh(oracle.dense_hamiltonian(cl))
    v0 = inputs.lanczos_start(cl.nd, 3)
    _, _, theta = binding.Operator(cl).lanczos(k, torch.from_numpy(v0).cuda())
    n, top = cl.nd, np.abs(lam).max()
    low, high = (lam[:k] - theta).max() / top, (theta - lam[n - k:]).max() / top
    print(f"k {k} of {n}: interlacing exceeded by {max(low, high):.2e}", flush=True)
    assert max(low, high) <= 1e-11
