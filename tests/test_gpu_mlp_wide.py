"""The fused forward pass of ensembles with more features than its workgroup
holds at a time (320): the features pass through LDS in pieces.

* against the float64 MLP oracle at one feature more than a piece, a whole
  number of pieces, a last piece of one fragment (16 features), one and two
  column tiles per wave and idle waves, ragged row tiles, with the tolerances
  of test_gpu_sur.py;
* features that are zero add exact zeros: a wide engine fed with a narrow
  engine's features and zeros gives that engine's outputs to the bit."""
import numpy as np
import pytest

from oracle import mlp_oracle as mo
from test_gpu_sur import _close, _cuda, _members

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("E,nin,nh,nout,B", [(2, 321, 32, 2, 1), (1, 640, 288, 3, 65), (1, 656, 256, 3, 33), (2, 700, 512, 3, 40),
                                             (1, 1500, 96, 32, 70), (2, 320, 64, 3, 31)])
def test_wide_forward_matches_oracle(E, nin, nh, nout, B):
    sur = _cuda()
    print(f"wide forward E={E} nin={nin} nh={nh} nout={nout} B={B}", flush=True)
    M = _members(E, nin, nh, nout, seed=nin + nh)
    X = np.random.default_rng(B).normal(size=(B, nin)).astype(np.float32)
    s = sur.Surrogate(M, nin, nh, nout, max_batch=B)
    Y = s.forward(torch.from_numpy(X).cuda()).cpu().numpy()
    Z = torch.empty((E, B, nout), dtype=torch.float32, device="cuda")
    s.forward_static(torch.from_numpy(X).cuda(), Z)
    s.close()
    for e in range(E):
        _close(Y[e], mo.forward(M[e], X.astype(np.float64))[0], f"Y member {e}")
    assert np.array_equal(Z.cpu().numpy(), Y)


@pytest.mark.parametrize("nh", [32, 160, 256, 320])
def test_zero_features_change_nothing(nh):
    sur = _cuda()
    print(f"zero features nh={nh}", flush=True)
    nin, more, B = 300, 500, 77
    M = _members(2, nin, nh, 3, seed=nh)
    rng = np.random.default_rng(nh)
    wide = [dict(m, W1=np.concatenate([m["W1"], rng.normal(size=(more, nh)).astype(np.float32)])) for m in M]
    X = rng.normal(size=(B, nin)).astype(np.float32)
    a = sur.Surrogate(M, nin, nh, 3, max_batch=B)
    b = sur.Surrogate(wide, nin + more, nh, 3, max_batch=B)
    x = torch.from_numpy(X).cuda()
    z = torch.cat([x, torch.zeros((B, more), device="cuda")], dim=1)
    assert torch.equal(a.forward(x), b.forward(z))
    a.close()
    b.close()
