"""The gauge force on lattices whose 16-site workgroups straddle lines and planes (the smallest lattice is one workgroup),
the link update over norms that need no and several squarings, and the context's links after a trajectory."""
import numpy as np
import pytest
import torch

from gpu_common import M0, ctx_and_oracle, rand5, relerr
from paper_1710_09621_amd import inputs as IN

pytestmark = pytest.mark.gpu


def _setup(dims, eps, seed):
    from paper_1710_09621_amd import eofa as E
    print(f"[gpu] gauge kernels dims={dims} eps={eps}", flush=True)
    Lx, Ly, Lz, Lt = dims
    U = IN.gauge_links(dims, eps, seed).reshape(Lt, Lz, Ly, Lx, 4, 3, 3)
    return E.Context(dims, 4, M0, IN.optimal_omega(4)), U


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 2, 4, 2), (2, 6, 2, 10), (10, 4, 2, 6), (16, 2, 2, 4)], ids=str)
def test_gauge_force_ragged(dims):
    from oracle import hmc as H
    ctx, U = _setup(dims, 0.8, 41)
    F = ctx.gauge_force(U, 6.2).cpu().numpy()
    Fr = H.gauge_force(U, dims, 6.2)
    assert np.abs(F - Fr).max() <= 1e-12 * np.abs(Fr).max()


@pytest.mark.parametrize("tau", [1e-3, 0.3, 4.0, 30.0])
def test_link_update(tau):
    """beta = 0 and one step: U <- exp(i tau P / 2) U twice.  Every squaring doubles the rounding of a 3 x 3
    exponential (a few 1e-16); |tau P / 2|_F <= 100 takes at most 8, so 1e-12 leaves a margin of ten."""
    from oracle import hmc as H
    dims = (2, 6, 4, 2)
    ctx, U = _setup(dims, 0.5, 42)
    Lx, Ly, Lz, Lt = dims
    P = np.random.default_rng(43).standard_normal((4, Lt, Lz, Ly, Lx, 8))
    Ug, Pg = torch.from_numpy(U.copy()).cuda(), torch.from_numpy(P.copy()).cuda()
    ctx.set_gauge(U)
    info = ctx.md_trajectory(Ug, Pg, [], 0.0, tau, [1])
    ref = H.update_links(H.update_links(U, dims, P, tau / 2), dims, P, tau / 2)
    assert info["link_updates"] == 2 and np.array_equal(Pg.cpu().numpy(), P)
    assert np.abs(Ug.cpu().numpy() - np.asarray(ref).reshape(U.shape)).max() <= 1e-12


def test_context_follows_the_links():
    """After a pure-gauge trajectory, whose gauge force never needs them, the context's packed links are those of
    the end point; after a rejected one those of the start."""
    from paper_1710_09621_amd import eofa as E
    dims, Ns = (4, 4, 2, 6), 8
    ctx, lat = ctx_and_oracle(dims, Ns, seed=44)
    print(f"[gpu] context links after a trajectory dims={dims}", flush=True)
    Lx, Ly, Lz, Lt = dims
    U = torch.from_numpy(IN.gauge_links(dims, 0.5, 44).reshape(Lt, Lz, Ly, Lx, 4, 3, 3)).cuda()
    P = torch.from_numpy(np.random.default_rng(45).standard_normal((4, Lt, Lz, Ly, Lx, 8))).cuda()
    x = rand5(lat, 46)
    start = U.clone()
    ctx.md_trajectory(U, P, [], 6.0, 0.5, [4])
    moved = ctx.apply("DT", x, 0.1, 0.3)
    other = E.Context(dims, Ns, M0, IN.optimal_omega(Ns))
    other.set_gauge(U)
    assert torch.equal(moved, other.apply("DT", x, 0.1, 0.3))
    assert relerr(moved, lat.dt(x, 0.1, 0.3)) > 1e-3  # the links did move
    # one coarse step from hot momenta: dH is far above the log of any accepted draw
    U.copy_(start)
    info = ctx.md_trajectory(U, 20.0 * P, [], 50.0, 2.0, [1], metropolis_u=0.999)
    assert info["accepted"] == 0 and torch.equal(U, start)
    assert relerr(ctx.apply("DT", x, 0.1, 0.3), lat.dt(x, 0.1, 0.3)) < 1e-12
