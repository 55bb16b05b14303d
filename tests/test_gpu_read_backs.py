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
