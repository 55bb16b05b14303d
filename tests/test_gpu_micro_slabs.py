"""The micro engine's launch rules at their edges: slabs of the binning (1024
particles each, at most 2048 in LDS, more through global memory), the wide
force kernel (at most 256 work blocks of 256 particles) against the one-lane
kernel, its spill path (a stencil row with more than 12 neighbours), windows of
partial sums and the default box groups.  The reference is the same engine
with one box per call, another slab width or the launches of single steps: all
routes add in the same order, so results agree to the bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _micro():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2512_13267_amd import inputs, micro
    return inputs, micro


def _params(inputs):
    return dict(inputs.lhmm_boxes(1, n_particles=300, polymer_fraction=0.0, seed_k=1).params)


def _run(m, G, s, c, steps, calls=1):
    m.set_state(s, c)
    out = [m.step(G, steps).cpu().numpy() for _ in range(calls)]
    st = m.get_state(with_forces=True)
    return out + [st[0], st[1], st[2], st[4]]


def _same(a, b, what):
    for x, y in zip(a, b):
        assert np.isfinite(x).all() and np.array_equal(x, y), what


def _state(rng, n, squeeze):
    s = rng.random((n, 3))
    if squeeze < 1.0:  # most particles in a slice of the box along the slab direction
        k = int(0.8 * n)
        s[:k, 0] *= squeeze
    return s, rng.normal(size=(n, 3))


@pytest.mark.parametrize("precision,n,edge,squeeze", [("fp32", 1024, 7.0, 1.0), ("fp32", 1025, 7.0, 1.0),
                                                      ("fp64", 2049, 9.0, 1.0), ("fp32", 6000, 13.0, 0.2),
                                                      ("fp64", 2600, 9.6, 0.12), ("fp32", 30, 14.0, 1.0)])
def test_slab_edges_do_not_change_results(precision, n, edge, squeeze):
    """Slab counts 1 / 2 / 3, slabs beyond their LDS (squeezed), cells mostly
    empty (n = 30): other slab widths and unfused steps give the same bits.
    Soft forces: the squeezed start stays finite over a few steps."""
    inputs, micro = _micro()
    print(f"slabs {precision} n={n} squeeze={squeeze}", flush=True)
    p = _params(inputs)
    p["dt"] = 1e-4
    s, c = _state(np.random.default_rng(n), n, squeeze)
    G = torch.tensor(inputs.planar_gradient(0.1, -0.05, 0.07).reshape(1, 9), dtype=torch.float64, device="cuda")
    ref = None
    for fuse, split in ((1, 0), (1, 256), (0, 0), (0, 700)):
        m = micro.Micro(p, [(n, 0, np.diag([edge] * 3))], precision=precision)
        m.set_config(fuse_bin=fuse, bin_split=split)
        got = _run(m, G, s, c, 5, calls=2)
        m.close()
        ref = ref or got
        _same(ref, got, (fuse, split))


@pytest.mark.parametrize("components", [False, True])
@pytest.mark.parametrize("nblk", [256, 257])
def test_wide_and_one_lane_forces_agree(nblk, components):
    """One box alone (wide kernel) equals the same box in a launch of 256 (wide)
    and 257 work blocks (one lane per particle); a dense spot takes the wide
    kernel's spill path."""
    inputs, micro = _micro()
    print(f"wide against one lane, {nblk} blocks, components={components}", flush=True)
    p = _params(inputs)
    p["dt"] = 1e-4
    rng = np.random.default_rng(nblk)
    n0, fill = 700, (nblk - 3) * 256
    h = np.diag([6.2, 6.2, 6.2])
    hb = np.diag([25.0] * 3)
    s0, c0 = _state(rng, n0, 1.0)
    s0[:60] = 0.5 + 0.02 * rng.random((60, 3))  # 60 neighbours within one cutoff
    sb, cb = _state(rng, fill, 1.0)
    L = inputs.planar_gradient(0.1, -0.05, 0.07).reshape(1, 9)
    one = torch.tensor(L, dtype=torch.float64, device="cuda")
    two = torch.tensor(np.concatenate([L, 0 * L]), dtype=torch.float64, device="cuda")
    a = micro.Micro(p, [(n0, 0, h, 5)], components=components)
    b = micro.Micro(p, [(n0, 0, h, 5), (fill, 0, hb, 6)], components=components)
    a.set_state(s0, c0)
    b.set_state(np.concatenate([s0, sb]), np.concatenate([c0, cb]))
    for steps in (1, 6):
        x, y = a.step(one, steps).cpu().numpy(), b.step(two, steps).cpu().numpy()
        assert np.isfinite(x).all() and np.array_equal(x[0], y[0]), steps
        if components:
            assert np.array_equal(a.components()[0], b.components()[0])
    for q in (0, 1):
        assert np.array_equal(a.get_state()[q], b.get_state()[q][:n0])
    a.close()
    b.close()


def test_windows_and_chunks_do_not_change_results():
    """Calls longer than a window of partial sums (50 steps), odd and even
    chunks and single steps accumulate the same sums."""
    inputs, micro = _micro()
    wl = inputs.lhmm_boxes(3, n_particles=400, polymer_fraction=0.2, seed_k=3)
    G = torch.tensor(np.stack([inputs.planar_gradient(0.1, 0.05, 0.0)] * 3).reshape(3, 9), dtype=torch.float64,
                     device="cuda")
    ref = None
    for chunk, fuse in ((50, 1), (51, 1), (200, 1), (7, 1), (50, 0)):
        print(f"windows chunk={chunk} fuse={fuse}", flush=True)
        m = micro.from_workload(wl)
        m.set_config(graph_chunk=chunk, fuse_bin=fuse)
        out = m.step(G, 117).cpu().numpy()
        st = m.get_state()
        pairs = m.pair_total()
        m.close()
        got = [out, st[0], st[1], st[2], pairs]
        ref = ref or got
        _same(ref, got, (chunk, fuse))


def test_default_groups_follow_the_size():
    inputs, micro = _micro()
    p = _params(inputs)
    for n_box, n, groups in ((3, 300, 1), (4, 255 * 256, 1), (4, 256 * 256, 2), (14, 256 * 256, 3)):
        m = micro.Micro(p, [(n, 0, np.diag([25.0] * 3))] * n_box)
        assert m.config()["groups"] == groups
        m.close()
