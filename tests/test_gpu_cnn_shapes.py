"""Network forward, loss and gradient on the shapes at the edges of the kernels' tiles (a compressed x extent of 1, odd
ones and ones above 8, the smallest y and z, Ns = 8, 16 and 32), against the CPU reference with the budget of
test_gpu_cnn.py: BF16 roundings that the summation order puts on another side, a few u / 10 in relative L2."""
import numpy as np
import pytest
import torch

from gpu_common import ctx_and_oracle, rand5
from oracle import cnn_ref as R
from paper_1710_09621_amd import inputs as IN

pytestmark = pytest.mark.gpu

TOL = 1e-2  # forward and loss; three times that for gradients, which pass through the forward's roundings
CASES = [((2, 4, 2, 6), 8), ((6, 2, 4, 2), 16), ((4, 2, 2, 4), 32), ((10, 6, 2, 4), 16), ((18, 2, 2, 2), 8), ((22, 2, 2, 4), 16)]


def _l2(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("dims,Ns", CASES, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_forward_and_gradient(dims, Ns, relu):
    print(f"[gpu] cnn shapes dims={dims} Ns={Ns} relu={relu}", flush=True)
    ctx, lat = ctx_and_oracle(dims, Ns)
    p = IN.cnn_params(51, scale=1.5)
    ctx.set_precond(p, relu=relu)
    rho, e = rand5(lat, 52), rand5(lat, 53)
    Lx, Ly, Lz, Lt = dims
    t, z, y, x = np.indices((Lt, Lz, Ly, Lx))
    odd = ((x + y + z + t) & 1).astype(bool)
    got = ctx.cnn_apply(torch.as_tensor(rho)).cpu().numpy()
    assert np.all(got[:, ~odd] == 0)
    assert _l2(got[:, odd], R.apply(rho, dims, p, relu=relu, bf16=True)[:, odd]) < TOL
    L, g = ctx.cnn_train_step(torch.as_tensor(rho), torch.as_tensor(e), lr=0.0, want_grad=True)
    Lr, gr = R.loss_and_grad(rho, e, dims, p, relu=relu, bf16=True)
    assert abs(L - Lr) < TOL * Lr
    for l in range(R.LAYERS):
        w, b = slice(l * R.LSZ, l * R.LSZ + R.WSZ), slice(l * R.LSZ + R.WSZ, (l + 1) * R.LSZ)
        assert _l2(g[w], gr[w]) < 3 * TOL and _l2(g[b], gr[b]) < 3 * TOL, l
        Wg = g[w].reshape(81, 32, 32)
        assert np.all(Wg[:, R.COUT[l]:, :] == 0) and np.all(Wg[:, :, R.CIN[l]:] == 0)
