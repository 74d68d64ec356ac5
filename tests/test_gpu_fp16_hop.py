"""The FP16-column hops themselves: their solves may not be repaired by the FP64 defect correction, and two CG iterations
are compared with those of FP32 storage element by element.  Below and above the split form's limit of 49,152
(site, s) lanes, at every Ns that FP16 columns have."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_common import ctx_and_oracle, rand5

pytestmark = pytest.mark.gpu

# k_hop_split: 16384, 4096, 4096 lanes; k_hop_mr: 65536 each; ragged last workgroup of either
CASES = [((8, 8, 8, 8), 8), ((4, 4, 4, 8), 16), ((4, 4, 4, 4), 32), ((8, 8, 8, 32), 8), ((8, 8, 8, 16), 16),
         ((8, 8, 8, 8), 32), ((6, 2, 2, 6), 8), ((10, 6, 12, 14), 16)]
IDS = lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c)  # noqa: E731
U16 = 2.0 ** -12  # rounding of a component relative to the largest of its column


@pytest.mark.parametrize("dims,Ns", CASES, ids=IDS)
def test_solve_needs_no_repair(dims, Ns):
    """The columns are rounded by 2.4e-4, so a cycle of the recurrence ends at a tenth of its start's residual up to a
    percent or so, and 1e-10 / 4 takes 11 replacements: twice that is the bound.  An operator that is wrong by a sign, a
    rotation or a norm stalls instead, or needs the FP64 solver."""
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] fp16 hop, solves dims={dims} Ns={Ns}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    bs = [torch.from_numpy(rand5(lat, 90 + j)).cuda() for j in range(3)]
    masses = [(0.05, 0.3), (1.0, 0.1), (0.2, 0.2)]
    P = E.params(tol=1e-10, prec=E.MIXED_FP16)
    got = [ctx.solve_ht(b, *m, P)[1] for b, m in zip(bs, masses)] + [i for _, i in ctx.solve_ht_batch(masses, bs, P)]
    want = [ctx.solve_ht(b, *m, E.params(tol=1e-10))[1] for b, m in zip(bs, masses)] * 2
    for g, w in zip(got, want):
        print(" ", g, w["iters"])
        assert g["fell_back"] == 0 and g["true_rel_resid"] <= 1e-10
        assert g["reliable_updates"] <= 22 and g["iters"] <= 2 * w["iters"]


def _two_iterations(ctx, E, b, mp, mm, prec):
    """x after exactly two CG iterations from zero (the solver reports that it has not converged)."""
    p = E.params(tol=1e-10, prec=prec, max_iter=2)
    x, info = torch.empty_like(b), E.SolveInfo()
    ctx._prep_ws(p)
    st = ctx.lib.eofa_solve_ht(ctx.h, mp, mm, C.c_void_p(b.data_ptr()), C.c_void_p(x.data_ptr()), C.byref(p), C.byref(info))
    assert st != E.OK and info.iters == 2
    return x


@pytest.mark.parametrize("dims,Ns", CASES, ids=IDS)
def test_two_iterations_against_fp32(dims, Ns):
    """Two iterations apply the normal operator twice; every one of its four hops rounds its output column once, p once
    more, and the s-operators mix at most Ns columns with weights that add up to a few: some 10 roundings of a column's
    largest component, each amplified by a few.  100 roundings (2.4%) of the largest component bound every element; a wrong sign,
    rotation or norm in one direction changes elements by a tenth of it and more."""
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] fp16 hop, two iterations dims={dims} Ns={Ns}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    b = torch.from_numpy(rand5(lat, 95)).cuda()
    for m in ((0.05, 0.3), (1.0, 0.1)):
        x16, x32 = (_two_iterations(ctx, E, b, *m, pr).cpu().numpy() for pr in (E.MIXED_FP16, E.MIXED_FP32))
        err = np.abs(x16 - x32).max() / np.abs(x32).max()
        l2 = np.linalg.norm(x16 - x32) / np.linalg.norm(x32)
        print(f"  masses {m}: largest {err:.2e}, L2 {l2:.2e}")
        assert err < 100 * U16 and l2 < 20 * U16
