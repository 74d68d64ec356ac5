"""Who finishes a CG iteration's two reductions: the next hop and the x/p update while the partial sums are few, a
launch of their own above that; iterations are counted on the device, so blocks may run past the last one."""
import pytest
import torch

from gpu_common import ctx_and_oracle, rand5, relerr

pytestmark = pytest.mark.gpu

# Vh Ns = 32 (one workgroup), 131072 (finished in the x/p update in every precision), 262144 (a launch of its own)
CASES = [((2, 2, 2, 2), 4), ((8, 8, 8, 32), 16), ((8, 8, 16, 32), 16)]


@pytest.mark.parametrize("dims,Ns", CASES, ids=str)
@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_solve(dims, Ns, prec):
    """The same bits and counts whether the host looks after each iteration or after seven, eager or captured; the
    solution against the operator.  1e-10 is the requested residual, 1e-11 the rounding of its own evaluation."""
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] reductions dims={dims} Ns={Ns} prec={prec}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    b = torch.from_numpy(rand5(lat, 41)).cuda()
    ref = None
    for kw in (dict(check_every=1), dict(check_every=7), dict(check_every=7, use_graph=1), dict()):
        x, info = ctx.solve_ht(b, 0.05, 0.3, E.params(tol=1e-10, prec=prec, **kw))
        assert info["true_rel_resid"] <= 1e-10
        res = (torch.linalg.vector_norm(b - ctx.apply("HT", x, 0.05, 0.3)) / torch.linalg.vector_norm(b)).item()
        assert abs(res - info["true_rel_resid"]) < 1e-11
        if ref is None:
            ref = (x.clone(), info["iters"])
        assert torch.equal(x, ref[0]) and info["iters"] == ref[1], kw


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("dims", [(8, 8, 8, 16), (8, 8, 16, 32)], ids=str)
def test_batch_equals_single(dims, prec):
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] reductions of a batch dims={dims} prec={prec}", flush=True)
    ctx, lat = ctx_and_oracle(dims, 16)
    bs = [torch.from_numpy(rand5(lat, 50 + j)).cuda() for j in range(3)]
    masses = [(0.05, 0.3), (1.0, 1.0), (0.1, 0.1)]  # the second converges first and is skipped from then on
    out = ctx.solve_ht_batch(masses, bs, E.params(tol=1e-11, prec=prec))
    for (mp, mm), b, (x, info) in zip(masses, bs, out):
        assert info["true_rel_resid"] <= 1e-11
        one, _ = ctx.solve_ht(b, mp, mm, E.params(tol=1e-11))
        assert relerr(x, one.cpu().numpy()) < 1e-8
