"""The density of blocks whose columns start inside a 16-byte unit: every offset
of the block's address, leading dimensions of every remainder, grids of less
than one unit, one wave (63 units) and a few waves, column counts around the
unrolled eight.  Reference: the same sum in NumPy FP64; both add the columns in
ascending order and differ by the rounding of g v v (2 or 3 roundings per term)
and of fused multiply-adds: 8 ns eps bounds it, terms being of one sign."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nd,ns", [(1, 1), (3, 9), (125, 8), (126, 7), (251, 17), (252, 8), (253, 3), (2017, 16)])
def test_density_offsets(nd, ns, dtype):
    from paper_1603_04334_amd import binding
    tdt = torch.float32 if dtype == "f32" else torch.float64
    rng = np.random.default_rng(nd + ns)
    h = 0.3
    for start in range(4):
        for pad in range(4):
            ld = nd + pad
            # rows of NaN before, between and behind the columns: nothing there may be used
            buf = np.full(start + ns * ld + 8, np.nan, dtype=np.float32 if dtype == "f32" else np.float64)
            vals = rng.standard_normal((ns, nd)).astype(buf.dtype)
            for c in range(ns):
                buf[start + c * ld:start + c * ld + nd] = vals[c]
            dev = torch.from_numpy(buf).cuda()
            psi = dev[start:].as_strided((ns, nd), (ld, 1))
            occ = np.sort(rng.uniform(0, 1, ns))[::-1].copy()
            rho = binding.density(psi, torch.from_numpy(occ).cuda(), h)
            torch.cuda.synchronize()
            ref = np.zeros(nd)
            for c in range(ns):
                ref += occ[c] * vals[c].astype(np.float64) ** 2
            ref *= 2.0 / h ** 3
            err = np.abs(rho.cpu().numpy() - ref).max() / ref.max()
            assert err <= 8 * ns * np.finfo(np.float64).eps, (start, pad, err)
