"""FP64 density of columns off the 16-byte grid (odd leading dimensions, blocks
that start on an odd value): grids around the 128 points of a wave, column
counts around the groups of two and eight, a grid that fills the chip, a block
beyond the last-level cache.

Sums of ns positive terms in FP64: relative error below ns eps against any
order, 2.3e-14 for 100 columns; the bound is 1e-13."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(nd, ns, pad, start):
    from paper_1603_04334_amd import binding
    g = torch.Generator(device="cuda").manual_seed(nd + ns)
    ld = nd + pad
    flat = torch.full((ns * ld + start + 1,), float("nan"), dtype=torch.float64, device="cuda")
    psi = torch.as_strided(flat, (ns, nd), (ld, 1), start)
    psi.copy_(torch.randn(ns, nd, generator=g, dtype=torch.float64, device="cuda"))
    occ = torch.rand(ns, generator=g, dtype=torch.float64, device="cuda")
    out = torch.full((nd + 2,), 7.0, dtype=torch.float64, device="cuda")
    binding.density(psi, occ, 0.4, out[1:-1])
    ref = (2.0 / 0.4 ** 3) * (occ[:, None] * psi * psi).sum(0)
    err = ((out[1:-1] - ref).abs() / ref).max().item()
    assert err <= 1e-13, (nd, ns, err)
    assert out[0] == 7.0 and out[-1] == 7.0


@pytest.mark.parametrize("nd", [1, 2, 63, 64, 65, 127, 128, 129, 255, 1001])
@pytest.mark.parametrize("ns", [1, 2, 3, 7, 8, 9, 17])
def test_small(nd, ns):
    _check(nd, ns, 1 - nd % 2, 0)  # odd leading dimension
    _check(nd, ns, nd % 2, 1)      # even one, the block starts on an odd value


@pytest.mark.parametrize("nd,ns", [(524287, 5), (524289, 9), (600001, 100), (2000001, 20)])
def test_large(nd, ns):
    _check(nd, ns, 1 - nd % 2, 0)
