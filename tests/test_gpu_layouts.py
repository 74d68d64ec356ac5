"""Canonical fields to the internal order and back, by size: cached, the canonical side streamed (above 256 MB), and the
half fields streamed too; eight consecutive sites that span several x rows."""
import numpy as np
import pytest
import torch

from gpu_common import ctx_and_oracle, relerr

pytestmark = pytest.mark.gpu

CASES = [((2, 2, 2, 2), 32), ((10, 2, 4, 2), 4), ((16, 16, 16, 32), 16), ((24, 16, 16, 32), 16)]


@pytest.mark.parametrize("dims,Ns", CASES, ids=str)
def test_pack_and_unpack(dims, Ns):
    """Dt moves both parities in and out, H_eo one of each: Dt at 64 sites against the oracle, and H_eo(x) + H_oe(x)
    the bits of H(x)."""
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] layouts dims={dims} Ns={Ns}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(lat.shape5, dtype=torch.complex128, device="cuda", generator=g)
    V = int(np.prod(dims))
    sites = np.unique(np.r_[0, V - 1, np.random.default_rng(6).integers(0, V, 62)]).astype(np.int64)
    ref = lat.dt_at(x.cpu().numpy(), 0.05, 0.3, sites)
    for prec, tol in ((E.FP64, 1e-12), (E.MIXED_FP32, 2e-6)):
        out = ctx.apply("DT", x, 0.05, 0.3, prec=prec).reshape(Ns, V, 12)[:, torch.from_numpy(sites).cuda()]
        assert relerr(out.transpose(0, 1).reshape(ref.shape), ref) < tol, prec
    assert torch.equal(ctx.apply("HOP_EO", x) + ctx.apply("HOP_OE", x), ctx.apply("HOP", x))


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (16, 8, 4, 16)], ids=str)
def test_hops_that_write_the_canonical_field(dims, prec):
    """The spin-split t-walk and the direction-split form write Dt, H_T, D_w and H to the canonical field themselves:
    the bits of the unsplit forms, whose results are moved."""
    print(f"[gpu] canonical output dims={dims} prec={prec}", flush=True)
    ctx, lat = ctx_and_oracle(dims, 16)
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randn(lat.shape5, dtype=torch.complex128, device="cuda", generator=g)
    ops = ["DT", "DT_DAG", "HT", "DW", "HOP"]
    cands = ctx.schedule_candidates(prec)
    by_mode = {s[0]: s for s in cands}
    assert 6 in by_mode and 5 in by_mode
    default = [ctx.apply(op, x, 0.05, 0.3, prec=prec) for op in ops]
    for mode in sorted(by_mode):
        ctx.set_schedule(by_mode[mode], prec)
        for op, ref in zip(ops, default):
            assert torch.equal(ctx.apply(op, x, 0.05, 0.3, prec=prec), ref), (mode, op)
