"""Every batch mode returns the bits of the standalone filter also for blocks
that the standalone filter gives to the row-pair kernels (large FP32 blocks,
FP64 grids that the one-row patches overhang): the batched modes step the same
sums on one-row patches."""
import pytest

import oracle
from paper_1603_04334_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# grid, columns, dtype, degree
JOBS = [((64, 64, 64), 40, "f32", 5), ((50, 83, 92), 12, "f64", 4), ((33, 70, 76), 64, "f32", 4)]


@pytest.mark.parametrize("mode", [0, 1, 2, 3, 4, 5])
def test_batch_bitwise_equals_rowpair_filter(mode):
    from paper_1603_04334_amd import binding
    binding.lib()
    jobs, refs, keep = [], [], []
    for n, ns, dtype, m in JOBS:
        cl = inputs.make_cluster(n, 0.45, 3, 8, 1, seed=sum(n), min_dist=0.0, margin=3.0)
        op = binding.Operator(cl)
        tdt, code = (torch.float32, binding.SPARC_F32) if dtype == "f32" else (torch.float64, binding.SPARC_F64)
        # neither the scalar nor a listed one-row patch
        assert op.step_config(code, ns)[:2] not in ((32, 16), (32, 32)), op.step_config(code, ns)
        X = inputs.device_orbitals(cl.nd, ns, sum(n), torch.float64).to(tdt).contiguous()
        Y = torch.empty_like(X)
        bounds = (-3.0, 1.5, oracle.upper_bound(cl))
        refs.append(op.cheb_filter(X, m, *bounds))
        jobs.append((op, X, Y, m, *bounds))
        keep.append(cl)
    torch.cuda.synchronize()
    batch = binding.Batch(jobs, mode=mode)
    for _ in range(2):
        for j in jobs:
            j[2].zero_()
        batch.run()
        torch.cuda.synchronize()
        assert batch.check() == 0
        for (op, X, Y, *_), ref in zip(jobs, refs):
            assert torch.equal(Y, ref), (op.cluster.n, mode, float((Y - ref).abs().max()))
    batch.close()
