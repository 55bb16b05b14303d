"""The allocation-free forward pass (lhmm_sur_forward_static) of an ensemble
that runs layer by layer (hidden = 544: its activations live in the library's
shared scratch) against lhmm_sur_forward of the same engine, whose activations
live in the engine's buffers: same kernels, weights and inputs, so the outputs
agree to the bit.  A later call with fewer rows must not see an earlier one's
scratch, nor one of another ensemble; batches beyond max_batch are served,
batches beyond the scratch refused before any launch."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_static_forward_of_layer_by_layer_ensembles():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2512_13267_amd import _lib, surrogate

    E, nin, nh, nout = 3, 33, 544, 3
    s = surrogate.Surrogate(surrogate.init_members(E, nin, nh, nout, seed=1), nin, nh, nout, max_batch=1500)
    other = surrogate.Surrogate(surrogate.init_members(2, 70, 576, 5, seed=2), 70, 576, 5, max_batch=400)
    g = torch.Generator(device="cpu")
    g.manual_seed(5)

    def pair(engine, B):
        print(f"static layers B={B} hidden={engine.n_hidden}", flush=True)
        X = torch.randn((B, engine.n_in), generator=g).cuda()
        Y = torch.full((engine.E, B, engine.n_out), float("nan"), device="cuda")
        engine.forward_static(X, Y)
        return X, Y

    for B in (1500, 999, 31, 1):
        X, Y = pair(s, B)
        assert torch.equal(Y, s.forward(X)) and torch.isfinite(Y).all(), B
        X, Y = pair(other, min(B, 400))
        assert torch.equal(Y, other.forward(X)), B
    B = 2000  # beyond max_batch, within the scratch
    X, Y = pair(s, B)
    ref = torch.cat([s.forward(X[k:k + 1000].contiguous()) for k in (0, 1000)], dim=1)
    assert torch.equal(Y, ref)
    most = 32 * ((32 << 20) // (32 * (2 * 64 + 4 * E * nh + 128 * E)))
    for B, ok in ((most - 32, True), (most + 32, False)):
        X = torch.zeros((B, nin), device="cuda")
        Y = torch.empty((E, B, nout), device="cuda")
        rc = _lib.lib().lhmm_sur_forward_static(s._h, ctypes.c_void_p(X.data_ptr()), B, ctypes.c_void_p(Y.data_ptr()))
        assert rc == (0 if ok else _lib.LHMM_ERR_ARG), B
    torch.cuda.synchronize()
    other.close()
    s.close()
