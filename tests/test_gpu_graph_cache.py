"""A program that cycles over many mass pairs with captured blocks captures each of them once."""
import pytest
import torch

from gpu_common import ctx_and_oracle, rand5

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["FP64", "MIXED_FP16"])
def test_graphs_of_many_mass_pairs_are_kept(prec):
    """60 sets of mass tables, every one with as many block lengths as the convergence rate asks for: the number of
    kept graphs never falls, a second pass adds none, and the solutions are those of the eager loop."""
    from paper_1710_09621_amd import eofa as E
    dims, Ns = (4, 4, 4, 4), 8
    print(f"[gpu] graph cache prec={prec}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    pr = getattr(E, prec)
    b = torch.from_numpy(rand5(lat, 81)).cuda()
    pairs = [(0.02 + 0.005 * k, 0.4) for k in range(60)]
    held, replays = [], []
    for p in range(2):
        for mp, mm in pairs:
            x, _ = ctx.solve_ht(b, mp, mm, E.params(tol=1e-10, prec=pr, use_graph=1))
            held.append(ctx.graph_stats()["cached"])
        replays.append(ctx.graph_stats()["replays"])
    assert held == sorted(held)
    assert held[-1] == held[len(pairs) - 1]
    assert replays[1] == 2 * replays[0]
    x0, _ = ctx.solve_ht(b, *pairs[-1], E.params(tol=1e-10, prec=pr))
    assert torch.equal(x, x0)
