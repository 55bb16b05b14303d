"""What the engines' synchronous reads return and wait for."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")


@pytest.mark.parametrize("n,boxes", [(700, 2), (2000, 40)])  # wide and one-lane force kernel
def test_a_force_evaluation_leaves_the_last_calls_pair_counts(n, boxes):
    """pair_counts is the count over the steps of the last step call."""
    _gpu()
    from paper_2512_13267_amd import inputs, micro

    print(f"pair counts after forces, {boxes} boxes of {n}", flush=True)
    wl = inputs.lhmm_boxes(boxes, n_particles=n, polymer_fraction=0.1, seed_k=17)
    G = np.stack([inputs.planar_gradient(0.1, -0.05, 0.07)] * boxes).reshape(boxes, 9)
    m = micro.from_workload(wl)
    m.step(torch.tensor(G, dtype=torch.float64, device="cuda"), 3)
    counts, total = m.pair_counts().copy(), m.pair_total().copy()
    assert (counts > 0).all()
    m.forces(G)
    assert np.array_equal(m.pair_counts(), counts)
    assert np.array_equal(m.pair_total(), total)
    m.close()


def test_a_read_of_nothing_waits_for_the_engine():
    """The reads are synchronous also where every destination is null."""
    _gpu()
    from paper_2512_13267_amd import _lib, inputs, lhmm, micro

    L = _lib.lib()
    mac = inputs.cylinder_array(n=16, force=2.0)
    nm = mac.r.shape[0] - mac.params["n_fixed"]
    m = micro.from_workload(inputs.lhmm_boxes(nm, n_particles=300, polymer_fraction=0.0, seed_k=3))
    G = torch.zeros((nm, 9), dtype=torch.float64, device="cuda")
    m.step(G, 2)
    s = lhmm.Sph(mac.params, mac.r, mac.v)
    h = lhmm.Hybrid(s, m, mode="dpd", k_micro=2)
    on = np.zeros(nm, dtype=np.uint32)
    reads = {
        "sph_get_state": lambda: L.lhmm_sph_get_state(s._h, None, None, None),
        "sph_coupling_state": lambda: L.lhmm_sph_coupling_state(s._h, None, None),
        "hybrid_state": lambda: L.lhmm_hybrid_state(h._h, None, on.ctypes.data_as(C.POINTER(C.c_uint32))),
        "hybrid_mean_stress": lambda: L.lhmm_hybrid_mean_stress(h._h, None, 0),
        "micro_get_state": lambda: L.lhmm_micro_get_state(m._h, None, None, None, None, None),
    }
    x = torch.randn((8192, 8192), device="cuda")
    y = x @ x
    torch.cuda.synchronize()
    for name, read in reads.items():
        print(f"read of nothing: {name}", flush=True)
        for _ in range(8):  # some 10 ms each
            torch.mm(x, x, out=y)
        done = torch.cuda.Event()
        done.record()
        m.step(G, 1)  # the micro engine's stream follows the caller's
        assert read() == 0
        assert done.query(), name
        torch.cuda.synchronize()
    h.close()
    s.close()
    m.close()


def test_weights_and_gradients_are_arrays_of_their_own():
    """Each tensor that get_weights and get_grads return can be kept, resized
    or dropped without the others."""
    _gpu()
    from paper_2512_13267_amd import surrogate

    E, nin, nh, nout = 2, 33, 64, 3
    s = surrogate.Surrogate(surrogate.init_members(E, nin, nh, nout, seed=2), nin, nh, nout, max_batch=8)
    s.train_step(torch.randn((8, nin), device="cuda"), torch.randn((8, nout), device="cuda"), 1e-3)
    for members in (s.get_weights(), s.get_grads()):
        for m in members:
            for k, x in m.items():
                assert x.base is None and x.flags.owndata and x.flags.c_contiguous, k
    s.close()
