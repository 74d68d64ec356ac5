"""Installed schedules are what runs: linear and tiled orders also where the direction-split form is the default,
the split form as a schedule of its own, and the default of every context among the autotuner's candidates.  The
operator has the same bits under every schedule; the reductions of CG blocks add in the order of the workgroups, so the
last bits of a row of them tell which schedule ran."""
import pytest
import torch

from gpu_common import M0, ctx_and_oracle, rand5, relerr
from paper_1710_09621_amd import inputs as IN

pytestmark = pytest.mark.gpu

SPLIT_LANES = 49152  # (site, s) lanes per parity up to which the split form exists


def _lanes(dims, Ns):
    return dims[0] * dims[1] * dims[2] * dims[3] // 2 * Ns


def _block(ctx, phi, sched=None):
    if sched is not None:
        ctx.set_schedule(sched)
    return [ctx.cg_block(+1, 0.05, 0.3, phi, n) for n in range(2, 34, 4)]


# at the split form's limit, just above it, no whole lines (linear orders only)
@pytest.mark.parametrize("dims,Ns", [((8, 8, 8, 8), 8), ((8, 8, 8, 12), 16), ((8, 8, 8, 14), 16), ((10, 6, 4, 6), 8)], ids=str)
def test_small_lattices_run_the_installed_schedule(dims, Ns):
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] schedules dims={dims} Ns={Ns}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    small = _lanes(dims, Ns) <= SPLIT_LANES
    phi = IN.gaussian_spinor(lat.shape4[:-2], 71)
    x = torch.from_numpy(rand5(lat, 72)).cuda()
    for prec in (E.FP64, E.MIXED_FP32, E.MIXED_FP16):
        cands = ctx.schedule_candidates(prec)
        assert [s for s in cands if s[0] == 2] == ([[2, 1, 1, 1, 1, 1, 0]] if small else []), prec
        if prec == E.MIXED_FP16:
            continue
        base = ctx.apply("DT", x, 0.05, 0.3, prec=prec)
        for s in (cands[0], cands[1], cands[-1]):
            ctx.set_schedule(s, prec)
            assert torch.equal(ctx.apply("DT", x, 0.05, 0.3, prec=prec), base), (prec, s)
    fresh, _ = ctx_and_oracle(dims, Ns)
    default, linear = _block(fresh, phi), _block(fresh, phi, cands[0])
    assert all(abs(a / b - 1) < 1e-8 for a, b in zip(linear, default))  # rounding, amplified by the iteration
    if small:  # four times as many workgroups, whose partial sums add in another order
        assert linear != default
        assert _block(fresh, phi, [2, 1, 1, 1, 1, 1, 0]) == default


# t-walk over half of the t extent (the whole one would leave half of the CUs idle), tiles, split form, ranges
@pytest.mark.parametrize("dims,Ns", [((16, 16, 16, 64), 16), ((16, 16, 16, 8), 16), ((8, 8, 8, 8), 8), ((10, 6, 12, 14), 16)],
                         ids=str)
def test_default_schedule_is_a_candidate(dims, Ns):
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] default schedule dims={dims} Ns={Ns}", flush=True)
    ctx = E.Context(dims, Ns, M0, IN.optimal_omega(Ns))
    ctx.set_gauge(IN.gauge_links(dims, 0.5, 73))
    phi = torch.randn(dims[::-1] + (4, 3), dtype=torch.complex128, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(74))
    default = _block(ctx, phi)
    assert any(_block(ctx, phi, s) == default for s in reversed(ctx.schedule_candidates(E.FP64)))


def test_autotuned_schedule_is_installed():
    from paper_1710_09621_amd import eofa as E
    dims, Ns = (8, 8, 8, 8), 8
    print(f"[gpu] autotuned schedule dims={dims} Ns={Ns}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    phi = IN.gaussian_spinor(lat.shape4[:-2], 75)
    for prec in (E.FP64, E.MIXED_FP32, E.MIXED_FP16):
        r = ctx.autotune(prec=prec)
        assert r["sched"] in ctx.schedule_candidates(prec) and r["best_ms"] <= r["base_ms"]
        if prec == E.FP64:
            got = _block(ctx, phi)
            assert got == _block(ctx, phi, r["sched"])


def test_fp64_default_is_tiled_at_ns32():
    """Its t-walk is the slower form on every lattice that has it (8 x 16 x 16 x 32: slower than linear order)."""
    from paper_1710_09621_amd import eofa as E
    dims, Ns = (8, 16, 16, 32), 32
    print(f"[gpu] default schedule dims={dims} Ns={Ns}", flush=True)
    ctx = E.Context(dims, Ns, M0, IN.optimal_omega(Ns))
    ctx.set_gauge(IN.gauge_links(dims, 0.5, 76))
    phi = torch.randn(dims[::-1] + (4, 3), dtype=torch.complex128, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(77))
    default = _block(ctx, phi)
    assert _block(ctx, phi, [1, 1, 4, 4, 8, 8, 0]) == default
    assert _block(ctx, phi, [5, 1, 4, 4, 32, 8, 0]) != default


# lines of 16 workgroups at Ns = 8: linear order in FP32 and FP16, tiles in FP64; batches at Ns = 32, where a single FP64
# solve is tiled and a batch linear
@pytest.mark.parametrize("dims,Ns", [((32, 32, 4, 4), 8), ((16, 8, 8, 6), 32)], ids=str)
@pytest.mark.parametrize("prec", [0, 1, 2], ids=["fp64", "fp32", "fp16"])
def test_batches_in_the_orders_of_the_rule(dims, Ns, prec):
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] batch orders dims={dims} Ns={Ns} prec={prec}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    masses = [(0.1 + 0.05 * j, 0.5) for j in range(3)]
    bs = [torch.from_numpy(rand5(lat, 78 + j)).cuda() for j in range(3)]
    for (mp, mm), b, (x, info) in zip(masses, bs, ctx.solve_ht_batch(masses, bs, E.params(tol=1e-11, prec=prec))):
        assert info["true_rel_resid"] <= 1e-11 and info["fell_back"] == 0
        one, _ = ctx.solve_ht(b, mp, mm, E.params(tol=1e-11))
        assert relerr(x, one.cpu().numpy()) < 1e-8
