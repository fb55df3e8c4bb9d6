"""Edges of the Rayleigh-Ritz projection and of the small rotations: block counts
that leave 1 to 4 block columns in the last tile, points short of a slice,
columns that start at any multiple of the element, grids below one slice.

The projection sums FP64 products in FP64, as the oracle does in another order:
N_d eps relative to |Y| |H Y| is below 1e-11 here, and the Ritz values of these
well-conditioned pencils inherit it; the bounds are those of the other
Rayleigh-Ritz tests (1e-9)."""
import numpy as np
import pytest

import oracle
from paper_1603_04334_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _op(cl):
    from paper_1603_04334_amd import binding
    return binding.Operator(cl)


def _check(cl, ns, dtype, pad):
    Y = inputs.round_to_f32(np.random.default_rng(ns).standard_normal((ns, cl.nd)))
    rt, _, Hs, Ms = oracle.rayleigh_ritz(cl, Y)
    big = torch.full((ns, cl.nd + pad), float("nan"), dtype=dtype, device="cuda")
    big[:, : cl.nd] = torch.from_numpy(Y).to(dtype).cuda()
    theta, Qt = _op(cl).rayleigh_ritz(big[:, : cl.nd])
    Q = Qt.cpu().numpy().T
    print(f"{cl.n} ns {ns} {dtype} pad {pad}: max |dtheta| {np.abs(theta - rt).max():.2e}", flush=True)
    assert np.abs(theta - rt).max() <= 1e-9 * max(1.0, np.abs(rt).max())
    assert np.abs(Q.T @ Ms @ Q - np.eye(ns)).max() < 1e-9
    assert np.abs(Hs @ Q - Ms @ Q * theta).max() < 1e-8 * max(1.0, np.abs(Hs).max())


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("ns", [15, 16, 17, 48, 49, 63, 65, 80, 81, 96, 97, 113, 128, 129, 200])
def test_projection_block_counts(ns, dtype):
    cl = inputs.make_cluster((17, 15, 21), 0.5, 2, 4, 1, seed=31, min_dist=0.0, margin=2.0)
    _check(cl, ns, dtype, ns % 4)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [(2, 3, 5), (1, 1, 32), (3, 11, 1), (4, 4, 4)])
def test_projection_short_grids(n, dtype):
    cl = inputs.free_cluster(n, 0.5)
    _check(cl, 5, dtype, 1)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("ns", [1, 3, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33, 50, 64, 65, 80, 81, 97, 113, 127, 128, 129,
                                160, 161, 192, 193, 224, 225])
def test_rotations(ns, dtype):
    """X Q on the device against FP64, a sum of ns products: ns eps |X| |Q|.
    Points short of a lane's, a wave's and a workgroup's share, columns that
    start on whole lines (704) and that do not; the values beside the columns
    stay as they were."""
    from paper_1603_04334_amd import binding
    for nd, pad in ((693, 0), (704, 0), (700, 4), (1, 0), (3, 2), (5, 0), (2113, 3)):
        rng = np.random.default_rng(1000 * ns + nd)
        X = inputs.round_to_f32(rng.standard_normal((ns, nd)))
        Q = inputs.round_to_f32(rng.standard_normal((ns, ns)))
        big = torch.full((ns, nd + pad), float("nan"), dtype=dtype, device="cuda")
        big[:, :nd] = torch.from_numpy(X).to(dtype).cuda()
        out = torch.full((ns, nd + pad), -7.0, dtype=dtype, device="cuda")
        binding.rotate(big[:, :nd], torch.from_numpy(Q).cuda(), out=out[:, :nd])
        got = out.double().cpu().numpy()
        eps = 2.0 ** -24 if dtype == torch.float32 else 2.0 ** -53
        bound = (ns + 1) * eps * (np.abs(Q) @ np.abs(X))
        assert (np.abs(got[:, :nd] - Q @ X) <= bound).all(), (nd, pad)
        assert (got[:, nd:] == -7.0).all(), (nd, pad)
