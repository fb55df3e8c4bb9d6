"""GPU parity of the electrostatic potential at the sizes where the solver's
kernels can go wrong: blocks of 4 x 4 x 4 nodes cut to 1, 2 and 3 nodes on each
axis, grids smaller than a block or the stencil, rows of one node (which the
single-vector step kernel does not take), odd rows, several patches and x-chunks.

Both sides run the same preconditioned CG in FP64 to ||r|| <= 1e-12 ||c - d||,
so iteration counts agree within one and the potentials to 1e-8 of their peak
(the residual tolerance times the condition number, at most 1e3 here, with
margin), as in the other parity tests of the solve."""
import numpy as np
import pytest

from oracle import poisson

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("n", [(3, 5, 9), (4, 4, 4), (9, 6, 1), (2, 13, 2), (5, 3, 35), (41, 18, 66), (22, 33, 31)])
def test_poisson_block_and_row_edges(n):
    from paper_1603_04334_amd import binding
    h = 0.4
    rng = np.random.default_rng(sum(n))
    x = [(np.arange(v) + 1) * h - 0.5 * (v + 1) * h for v in n]
    X, Y, Z = np.meshgrid(*x, indexing="ij")
    f = np.exp(-((X - 0.1) ** 2 + (Y + 0.2) ** 2 + Z ** 2) / 1.3) + 0.05 * rng.standard_normal(n)
    f = f.reshape(-1)
    P = binding.Poisson(n, h)
    phi, it, res, Q = P.solve(torch.from_numpy(f).cuda(), tol=TOL)
    torch.cuda.synchronize()
    ref, it_ref, _, _ = poisson.poisson_solve(n, h, 6, f, lmax=6, tol=TOL)
    err = np.abs(phi.cpu().numpy() - ref).max() / np.abs(ref).max()
    print(f"poisson {n}: iters {it} (oracle {it_ref}) resid {res:.2e} phi err {err:.2e}", flush=True)
    assert res <= TOL and abs(it - it_ref) <= 1 and err <= 1e-8
