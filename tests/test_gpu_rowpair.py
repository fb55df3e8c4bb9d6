"""GPU parity of the row-pair step kernels (two y rows per lane, patches fitted
to the grid, rows cut inside a 16-byte unit) against the oracle, at the sizes
where they can go wrong: every remainder of the row length, an odd number of y
rows, one and two patches along z, one and several along y, one and several
x-chunks, rows shorter than the stencil, padded leading dimensions that are no
multiple of the unit.  The library takes these kernels from 4e6 values per
block, so the columns of the small grids repeat a few distinct ones and only
those are compared; equal columns must come out bit for bit equal.

Tolerances as for the other filter kernels (per column, |Y - Y_ref| / |Y_ref|):
FP64 1e-12, FP32 5e-5 against the oracle fed the FP32-rounded inputs."""
import numpy as np
import pytest

import oracle
from paper_1603_04334_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # grid, columns, dtype, degree
    ((20, 46, 44), 220, "f32", 4),    # whole units, one patch
    ((17, 45, 49), 260, "f32", 4),    # 3 nodes short of whole units, odd rows
    ((14, 61, 50), 300, "f32", 3),    # 2 short
    ((14, 59, 51), 300, "f32", 3),    # 1 short
    ((9, 33, 165), 240, "f32", 3),    # two patches along z, cut rows
    ((11, 30, 164), 200, "f32", 3),   # two patches along z, whole units
    ((9, 200, 46), 130, "f32", 3),    # several patches along y
    ((70, 43, 47), 60, "f32", 3),     # several x-chunks
    ((15, 57, 49), 100, "f64", 3),    # FP64, cut rows
    ((9, 37, 101), 130, "f64", 3),    # FP64, two patches along z, cut rows
    ((60, 39, 31), 70, "f64", 3),     # FP64, narrow rows, several x-chunks
    ((13, 50, 68), 100, "f64", 3),    # FP64, whole units, patches that overhang otherwise
    ((3, 4, 5), 70000, "f32", 3),     # smaller than the stencil
]


@pytest.mark.parametrize("case", CASES, ids=["%s-%dx%d" % (c[2], c[1], c[0][2]) for c in CASES])
def test_rowpair_filter_and_h(case):
    from paper_1603_04334_amd import binding
    n, ns, dtype, m = case
    if min(n) > 8:
        cl = inputs.make_cluster(n, 0.5, 3, 6, 1, seed=sum(n), min_dist=0.0, margin=1.5)
    else:
        cl = inputs.free_cluster(n, 0.5, v0=-0.4)
    rng = np.random.default_rng(sum(n))
    distinct = rng.standard_normal((3, cl.nd))
    tdt, tol, ocl = (torch.float32, 5e-5, inputs.round_cluster_f32(cl)) if dtype == "f32" else (torch.float64, 1e-12, cl)
    if dtype == "f32":
        distinct = inputs.round_to_f32(distinct)
    op = binding.Operator(cl)
    # a leading dimension that is odd, so columns start inside a 16-byte unit
    pad = 3 if cl.nd % 2 == 0 else 2
    big = torch.zeros((ns, cl.nd + pad), dtype=tdt, device="cuda")
    big[:, : cl.nd] = torch.from_numpy(distinct).to(tdt).cuda()[torch.arange(ns, device="cuda") % 3]
    X = big[:, : cl.nd]
    outbig = torch.full((ns, cl.nd + pad + 2), 7.0, dtype=tdt, device="cuda")
    out = outbig[:, : cl.nd]
    a0, a, b = -3.0, 2.0, oracle.upper_bound(cl)
    for name, ref in (("h", oracle.h_apply(ocl, distinct)), ("filter", oracle.cheb_filter(ocl, distinct, m, a0, a, b))):
        if name == "h":
            op.h_apply(X, out)
        else:
            op.cheb_filter(X, m, a0, a, b, Y=out)
        torch.cuda.synchronize()
        for c in range(3):
            same = out[c::3]
            assert torch.equal(same, same[:1].expand_as(same)), (name, c)
        got = out[:3].double().cpu().numpy()
        err = (np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()
        config = op.step_config(binding.SPARC_F32 if dtype == "f32" else binding.SPARC_F64, ns)
        print(f"{name} {n} {dtype} config {config} err {err:.2e}", flush=True)
        assert config[:2] not in ((32, 16), (32, 32)), config  # neither the scalar nor the one-row patches
        assert err <= tol, name
        assert torch.all(outbig[:, cl.nd:] == 7.0)  # padding untouched
