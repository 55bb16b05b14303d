"""Micro-domains whose z extent is too small for the stencil (accepted, and
flagged LHMM_FLAG_CELL): the cells of a stencil row no longer span the cutoff,
so records past a row's range lie within it and must not be taken.  The wide
force kernel (a box alone) and the one-lane kernel (the same box in a launch
of more than 256 work blocks) scan the same candidates in the same order, so
forces, stresses and pair counts agree to the bit.

Boxes: two cells per cutoff along z (five cells of 0.4 rc) and one (70 x 70 x
2.2 rc, whose finer grid would pass the cell limit); also with stress
components kept apart and with the pruned stencil."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision,n,edges,components,prune", [("fp32", 1200, (9.0, 9.0, 2.0), False, 0),
                                                                ("fp64", 1200, (9.0, 9.0, 2.0), False, 0),
                                                                ("fp32", 9000, (70.0, 70.0, 2.2), False, 0),
                                                                ("fp32", 1200, (9.0, 9.0, 2.0), True, 0),
                                                                ("fp32", 1200, (9.0, 9.0, 2.0), False, 1)])
def test_flat_boxes_count_each_neighbour_once(precision, n, edges, components, prune):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2512_13267_amd import _lib, inputs, micro

    print(f"flat box {edges} n={n} {precision} components={components} prune={prune}", flush=True)
    p = dict(inputs.lhmm_boxes(1, n_particles=300, polymer_fraction=0.0, seed_k=1).params)
    p["dt"] = 1e-5
    rng = np.random.default_rng(n)
    fill = 260 * 256 - n
    s0, c0 = rng.random((n, 3)), rng.normal(size=(n, 3))
    sb, cb = rng.random((fill, 3)), rng.normal(size=(fill, 3))
    L = inputs.planar_gradient(0.1, -0.05, 0.07).reshape(1, 9)
    one = torch.tensor(L, dtype=torch.float64, device="cuda")
    two = torch.tensor(np.concatenate([L, 0 * L]), dtype=torch.float64, device="cuda")
    a = micro.Micro(p, [(n, 0, np.diag(edges), 5)], precision=precision, components=components)
    b = micro.Micro(p, [(n, 0, np.diag(edges), 5), (fill, 0, np.diag([25.0] * 3), 6)], precision=precision,
                    components=components)
    if prune:
        b.set_config(prune=1)
    a.set_state(s0, c0)
    b.set_state(np.concatenate([s0, sb]), np.concatenate([c0, cb]))
    for steps in (1, 4):
        x, y = a.step(one, steps).cpu().numpy(), b.step(two, steps).cpu().numpy()
        assert a.pair_counts()[0] == b.pair_counts()[0], steps
        assert np.isfinite(x).all() and np.array_equal(x[0], y[0]), steps
        if components:
            assert np.array_equal(a.components()[0], b.components()[0])
    for u, v in zip(a.get_state(with_forces=True), b.get_state(with_forces=True)):
        if np.ndim(u) == 2:
            assert np.array_equal(u, v[:n])
    assert a.flags()[0] & _lib.FLAG_CELL and b.flags()[0] & _lib.FLAG_CELL
    a.close()
    b.close()


@pytest.mark.parametrize("zsub", [2, 1])
def test_a_box_may_become_flat_by_its_state(zsub):
    """A state that is loaded may make a box too flat for its stencil, and a
    later one tall again: captured steps follow.  The reference is a fresh
    engine per state, alone (wide kernel)."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2512_13267_amd import inputs, micro

    print(f"box made flat by its state, zsub={zsub}", flush=True)
    p = dict(inputs.lhmm_boxes(1, n_particles=300, polymer_fraction=0.0, seed_k=1).params)
    p["dt"] = 1e-5
    rng = np.random.default_rng(zsub)
    edge, n = (9.0, 1200) if zsub == 2 else (70.0, 9000)
    fill = 260 * 256 - n
    s0, c0, sb, cb = rng.random((n, 3)), rng.normal(size=(n, 3)), rng.random((fill, 3)), rng.normal(size=(fill, 3))
    L = inputs.planar_gradient(0.1, -0.05, 0.07).reshape(1, 9)
    one = torch.tensor(L, dtype=torch.float64, device="cuda")
    two = torch.tensor(np.concatenate([L, 0 * L]), dtype=torch.float64, device="cuda")
    tall, big = np.diag([edge, edge, 3.5]), np.diag([25.0] * 3)
    b = micro.Micro(p, [(n, 0, tall, 5), (fill, 0, big, 6)])
    for z in (3.5, 2.1, 3.5, 2.4):
        h = np.diag([edge, edge, z])
        a = micro.Micro(p, [(n, 0, tall, 5)])
        a.set_state(s0, c0, h=h.reshape(1, 9))
        b.set_state(np.concatenate([s0, sb]), np.concatenate([c0, cb]), h=np.stack([h, big]).reshape(2, 9))
        x, y = a.step(one, 4).cpu().numpy(), b.step(two, 4).cpu().numpy()
        assert a.pair_counts()[0] == b.pair_counts()[0], z
        assert np.isfinite(x).all() and np.array_equal(x[0], y[0]), z
        a.close()
    b.close()
