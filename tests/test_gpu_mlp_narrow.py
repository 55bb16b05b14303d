"""The fused kernels' two-wave form (layers of one or two 32-column tiles, more
than 1024 workgroups of 32 rows and a member) against the eight-wave form: two
members together take the first, one member alone the second, with the same
sums in the same order, so outputs, losses, gradients and updated weights agree
to the bit.  513 row tiles, the last with one row; one tile and two; features
within a piece (192), beyond it (forward in pieces), and beyond the training
step's limit (320); and the float64 MLP oracle with the tolerances of
test_gpu_sur.py."""
import numpy as np
import pytest

from oracle import mlp_oracle as mo
from test_gpu_sur import _close, _cuda, _members

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nin,nh,nout", [(129, 32, 3), (40, 64, 32), (193, 64, 2), (330, 32, 3)])
def test_two_waves_agree_with_eight(nin, nh, nout):
    sur = _cuda()
    E, B = 2, 512 * 32 + 1
    print(f"two waves {nin}-{nh}-{nh}-{nout}", flush=True)
    M = _members(E, nin, nh, nout, seed=nin)
    rng = np.random.default_rng(nh)
    X = rng.normal(size=(B, nin)).astype(np.float32)
    T = rng.normal(size=(B, nout)).astype(np.float32)
    x, t = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()

    def all_of(members):
        s = sur.Surrogate(members, nin, nh, nout, max_batch=B)
        loss = torch.zeros(len(members), dtype=torch.float32, device="cuda")
        Y = s.forward(x).cpu().numpy()
        s.train_step(x, t, 1e-3, loss)
        G, W, L = s.get_grads(), s.get_weights(), loss.cpu().numpy()
        s.close()
        return Y, G, W, L

    Y, G, W, L = all_of(M)
    for e in range(E):
        y, g, w, lo = all_of([M[e]])
        assert np.array_equal(Y[e], y[0]) and L[e] == lo[0], e
        for k in g[0]:
            assert np.array_equal(G[e][k], g[0][k]) and np.array_equal(W[e][k], w[0][k]), (e, k)
    _close(Y[0], mo.forward(M[0], X.astype(np.float64))[0], "Y")
    lo, go, _ = mo.loss_and_grads(M[0], X.astype(np.float64), T.astype(np.float64))
    assert abs(L[0] - lo) < 1e-3 * lo
    for k in go:
        _close(G[0][k], go[k], f"grad {k}")
