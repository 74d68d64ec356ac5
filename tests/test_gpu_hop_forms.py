"""The forms of the hop that a launch takes by its size: direction-split below 49,152 (site, s) lanes over all systems,
one system after the other or side by side above it, and the workgroup order of a context that was never tuned."""
import pytest
import torch

from gpu_common import ctx_and_oracle, rand5, relerr

pytestmark = pytest.mark.gpu

# lanes per parity: at the split form's limit, just above it (unsplit, ragged last workgroup), and ragged at Ns = 32
CASES = [((8, 8, 8, 12), 16), ((8, 8, 8, 14), 16), ((6, 6, 2, 10), 32), ((10, 6, 12, 14), 8)]


@pytest.mark.parametrize("dims,Ns", CASES, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_operators_against_oracle(dims, Ns):
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] hop forms dims={dims} Ns={Ns}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    x = rand5(lat, 31)
    for op, ref in (("DT", lat.dt(x, 0.05, 0.3)), ("DT_DAG", lat.dt(x, 0.05, 0.3, dag=True)), ("HT", lat.ht(x, 0.05, 0.3))):
        assert relerr(ctx.apply(op, x, 0.05, 0.3), ref) < 1e-12, op
        assert relerr(ctx.apply(op, x, 0.05, 0.3, prec=E.MIXED_FP32), ref) < 2e-6, op


@pytest.mark.parametrize("Ns", [8, 16])
def test_split_form_bitwise_equals_twalk(Ns):
    """8^4 is below the split limit and has t-walk schedules: the same bits from both."""
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] split form against t-walk, 8^4 Ns={Ns}", flush=True)
    ctx, lat = ctx_and_oracle((8, 8, 8, 8), Ns)
    x = torch.from_numpy(rand5(lat, 32)).cuda()
    ops = ["DW", "HOP", "DT", "DT_DAG", "HT", "SCHUR", "SCHUR_DAG", "SCHUR_NORMAL", "DODWF", "DODWF_DAG", "HOP_EO"]
    for p in (E.FP64, E.MIXED_FP32):
        base = [ctx.apply(op, x, 0.05, 0.3, prec=p) for op in ops]
        tw = [s for s in ctx.schedule_candidates(p) if s[0] in (3, 5, 6)]
        assert tw
        ctx.set_schedule(tw[0], p)
        for op, b in zip(ops, base):
            assert torch.equal(ctx.apply(op, x, 0.05, 0.3, prec=p), b), (op, tw[0])


# 8^4 at Ns = 8: three systems are split, four and more run side by side; 8^3 x 16: side by side, then in pairs
@pytest.mark.parametrize("dims,Ns,n", [((8, 8, 8, 8), 8, 3), ((8, 8, 8, 8), 8, 4), ((8, 8, 8, 16), 16, 3), ((8, 8, 8, 16), 16, 8)],
                         ids=str)
@pytest.mark.parametrize("prec", [0, 1, 2], ids=["fp64", "fp32", "fp16"])
def test_batches_equal_single_solves(dims, Ns, n, prec):
    from paper_1710_09621_amd import eofa as E
    from paper_1710_09621_amd import inputs as IN
    print(f"[gpu] batch forms dims={dims} Ns={Ns} n={n} prec={prec}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    acts = ([(-1, 0.1, 0.1, 0.5), (+1, 0.1, 0.5, 1.0), (-1, 1.0, 0.5, 1.0), (+1, 0.2, 0.1, 0.5)] * 2)[:n]
    phis = [IN.gaussian_spinor(lat.shape4[:-2], 300 + j) for j in range(n)]
    res = ctx.chiral_action_batch(acts, phis, E.params(tol=1e-11, prec=prec, use_graph=1))
    for a, phi, r in zip(acts, phis, res):
        assert r.info[0]["true_rel_resid"] <= 1e-11
        one = ctx.chiral_action(*a, phi, E.params(tol=1e-11))
        assert relerr(r.out, one.out.cpu().numpy()) < 1e-8
        assert abs(r.S - one.S) < 1e-8 * abs(one.S)
