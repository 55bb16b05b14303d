"""GPU parity of the surrogate's fused kernels (csrc/lhmm_mlp.h) with the
float64 MLP oracle at the sizes where their tiling changes: one and two
column tiles per wave (the switch lies at 256 hidden units), idle waves, odd
tile counts of the weight gradients, one row, one more row than a tile, the
single-chunk and chunked weight gradients (the switch lies at 1024 rows); and
the first width that runs layer by layer instead (512 is the last fused one).

Tolerances are those of tests/test_gpu_sur.py: 1e-3 in the relative Frobenius
norm and 2^-6 of the scale for single values (one BF16 ulp, 2^-8, through a
product)."""
import numpy as np
import pytest

from oracle import mlp_oracle as mo
from test_gpu_sur import _close, _cuda, _data, _members, mo_layers

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("E,nin,nh,nout,B", [(2, 7, 32, 2, 1), (1, 129, 256, 3, 33), (2, 64, 288, 32, 65),
                                             (1, 129, 512, 3, 1023), (2, 33, 96, 3, 1025), (1, 40, 544, 3, 70)])
def test_fused_layers_match_oracle(E, nin, nh, nout, B):
    sur = _cuda()
    print(f"fused E={E} nin={nin} nh={nh} nout={nout} B={B}", flush=True)
    M = _members(E, nin, nh, nout, seed=50 + nh)
    X, T = _data(B, nin, max(nout, 1), seed=60 + B) if nout <= nin else (
        np.random.default_rng(60 + B).normal(size=(B, nin)).astype(np.float32),
        np.random.default_rng(61 + B).normal(size=(B, nout)).astype(np.float32))
    x, t = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    s = sur.Surrogate(M, nin, nh, nout, max_batch=B)
    Y = s.forward(x).cpu().numpy()
    Z = torch.empty((E, B, nout), dtype=torch.float32, device="cuda")
    s.forward_static(x, Z)
    assert np.array_equal(Z.cpu().numpy(), Y)
    loss = torch.zeros(E, dtype=torch.float32, device="cuda")
    s.train_step(x, t, 0.0, loss)
    G, L, W = s.get_grads(), loss.cpu().numpy(), s.get_weights()
    for e in range(E):
        ref, _ = mo.forward(M[e], X.astype(np.float64))
        _close(Y[e], ref, f"Y member {e}")
        lo, go, _ = mo.loss_and_grads(M[e], X.astype(np.float64), T.astype(np.float64))
        assert abs(L[e] - lo) < 1e-3 * lo, (e, L[e], lo)
        for k in mo_layers():
            _close(G[e][k], go[k], f"grad {k} member {e}")
            assert np.array_equal(W[e][k].astype(np.float64), M[e][k]), k  # lr = 0
    # the packed copies that an update writes serve the next pass
    s.train_step(x, t, 1e-3, loss)
    W = s.get_weights()
    Y = s.forward(x).cpu().numpy()
    for e in range(E):
        _close(Y[e], mo.forward({k: v.astype(np.float64) for k, v in W[e].items()}, X.astype(np.float64))[0], f"Y after {e}")
    s.close()
