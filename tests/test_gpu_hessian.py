"""GPU Hessian-vector products (§5.2) vs the FP64 oracle, and the identities
a Hessian must satisfy at sizes the oracle does not reach.

Tolerance: the FP32 second-order pass is compared with the FP64 oracle by the
max-abs error over all atoms relative to the largest entry of the reference
product, <= 2e-5 (measured: at most 1.2e-6; the errors are printed)."""
import numpy as np
import pytest

import synth
from oracle import model as om
from tests.gpu_util import device, model, say, to_dev

pytestmark = pytest.mark.gpu

REL = 2e-5


def _graph(m, b, skin=0.0):
    pos, sp = to_dev(b)
    cfg = synth.ModelConfig.from_json(m.config_json)
    return m.build_graph(b.offsets, pos, sp, b.cell, b.pbc, cfg.cutoff, skin), pos


def _hv(m, b, v, skin=0.0):
    import torch
    g, pos = _graph(m, b, skin)
    hv = m.hessian_vector(g, pos, torch.tensor(v, dtype=torch.float32, device=device()))
    torch.cuda.synchronize()
    return hv.cpu().numpy().astype(np.float64)


def _check(hv, ref, what):
    err = np.abs(hv - ref).max()
    scale = np.abs(ref).max()
    say(f"  {what}: max err {err:.2e} of max |Hv| {scale:.2e} ({err / scale:.2e})")
    assert err <= REL * scale, (err, scale)


def test_tiny_cluster_against_oracle():
    cfg, b = synth.tiny_config()
    w = synth.model_weights(cfg, 1)
    m = model(cfg, 1)
    rng = np.random.default_rng(111)
    for k in range(2):
        v = rng.normal(size=b.pos.shape)
        _check(_hv(m, b, v), om.hessian_vector(om.Model(cfg, w), b, v), f"tiny v{k}")


def test_packed_periodic_batch_against_oracle():
    cfg, b, _, _ = synth.differentiation_config(4, 20, 90)
    m = model(cfg, 3)
    v = np.random.default_rng(112).normal(size=b.pos.shape)
    ref = om.hessian_vector(om.Model(cfg, synth.model_weights(cfg, 3)), b, v)
    _check(_hv(m, b, v, skin=0.5), ref, f"packed N={b.n_atoms}")


def test_sampled_rows_and_full_hessian_against_oracle():
    # a batch of small open molecules, as in the paper's Hessian study
    cfg = synth.ModelConfig(lmax=3, channels=32, layers=2, n_species=4, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0))
    rng = np.random.default_rng(113)
    parts = [synth.open_box(n, 4, rng) for n in (9, 12, 7)]
    b = synth.concat(parts)
    m = model(cfg, 114)
    om_m = om.Model(cfg, synth.model_weights(cfg, 114))
    g, pos = _graph(m, b)
    rows = np.array([[3, 0, 6], [8, 11, 2]])
    R = m.hessian_rows(g, pos, rows).cpu().numpy().astype(np.float64)
    for r in range(2):
        for a in range(3):
            v = np.zeros(b.pos.shape)
            v[b.offsets[:-1] + rows[r], a] = 1.0
            _check(R[r, a], om.hessian_vector(om_m, b, v), f"row {r} axis {a}")
    H = [h.cpu().numpy().astype(np.float64) for h in m.hessian(g, pos)]
    for s, p in enumerate(parts):
        n = p.n_atoms
        Href = np.zeros((3 * n, 3 * n))
        for k in range(3 * n):
            e = np.zeros(3 * n)
            e[k] = 1.0
            Href[:, k] = om.hessian_vector(om_m, p, e.reshape(n, 3)).reshape(-1)
        err = np.abs(H[s] - Href).max()
        say(f"  full Hessian of structure {s}: max err {err:.2e} of {np.abs(Href).max():.2e}")
        assert err <= REL * np.abs(Href).max()
        assert np.abs(H[s] - H[s].T).max() <= REL * np.abs(Href).max()


def test_identities_on_a_large_open_cluster():
    # translation: H t = 0; rotation: H (w x r) = -(w x F); symmetry u.Hv = v.Hu
    import torch
    cfg = synth.ModelConfig(lmax=3, channels=64, layers=2, n_species=4, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0))
    b = synth.open_box(1500, 4, np.random.default_rng(115))
    m = model(cfg, 116)
    g, pos = _graph(m, b)
    _, F = m.energy_forces(g, pos)[:2]
    F = F.cpu().numpy().astype(np.float64)
    dev = device()

    def hv(v):
        out = m.hessian_vector(g, pos, torch.tensor(v, dtype=torch.float32, device=dev))
        return out.cpu().numpy().astype(np.float64)
    rng = np.random.default_rng(117)
    u, v = rng.normal(size=b.pos.shape), rng.normal(size=b.pos.shape)
    Hu, Hv = hv(u), hv(v)
    scale = np.abs(Hv).max()
    c = b.pos.mean(0)
    w = np.array([0.3, -0.5, 0.8])
    Ht = hv(np.tile([1.0, -2.0, 0.5], (b.n_atoms, 1)))
    Hr = hv(np.cross(w, b.pos - c))
    say(f"  |H t| {np.abs(Ht).max():.2e}, rotation {np.abs(Hr + np.cross(w, F)).max():.2e}, "
        f"scale {scale:.2e}")
    assert np.abs(Ht).max() <= REL * scale
    # (H (w x (r - c)) = -(w x F) + H (w x c) and H (w x c) = 0 (a translation)
    assert np.abs(Hr + np.cross(w, F)).max() <= REL * max(scale, np.abs(F).max())
    a1, a2 = np.sum(u * Hv), np.sum(v * Hu)
    assert abs(a1 - a2) <= 1e-4 * np.sqrt(np.sum(u * Hu) ** 2 + np.sum(v * Hv) ** 2 + a1 ** 2)


def test_unsupported_models_are_rejected():
    import torch
    import paper_2605_22698_amd as e3
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=2, n_species=3, cutoff=5.0, avg_neighbors=10.0,
                            coulomb=True)
    m = model(cfg, 118)
    b = synth.open_box(12, 3, np.random.default_rng(119))
    g, pos = _graph(m, b)
    with pytest.raises(e3.E3miError):
        m.hessian_vector(g, pos, torch.zeros((12, 3), device=device()))


@pytest.mark.parametrize("lmax,C,layers", [(2, 32, 2), (3, 64, 3)])
def test_product_block_against_oracle(lmax, C, layers):
    # the product block's tangent and its reverse (correlation 2): every layer
    # with every order of A; the middle layer of three has all output orders
    cfg = synth.ModelConfig(lmax=lmax, channels=C, layers=layers, n_species=4, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0), correlation=2)
    rng = np.random.default_rng(120 + layers)
    b = synth.concat([synth.jittered_lattice(n, 0.1, 0.3, 4, rng) for n in (40, 27)])
    m = model(cfg, 121)
    w = synth.model_weights(cfg, 121)
    for k in range(2):
        v = rng.normal(size=b.pos.shape)
        _check(_hv(m, b, v, skin=0.5), om.hessian_vector(om.Model(cfg, w), b, v),
               f"product block lmax {lmax} C {C} layers {layers} v{k}")


@pytest.mark.parametrize("correlation", [1, 2])
def test_isolated_atom_and_empty_structure(correlation):
    # degenerate inputs of the second-order pass: an empty structure, and a
    # structure with an isolated atom beside a small cluster; the Hessian-vector
    # product against the oracle (zero rows for the isolated atom) and the
    # parameter gradient finite
    import torch
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=2, n_species=3, cutoff=5.0, avg_neighbors=10.0,
                            correlation=correlation)
    rng = np.random.default_rng(150)
    cl = synth.uniform_cluster(8, 5.0, 1.0, 3, rng)
    pos = np.concatenate([cl.pos, [[40.0, 40.0, 40.0]]])
    sp = np.concatenate([cl.species, [1]]).astype(np.int32)
    cells = (np.eye(3) * 100.0)[None].repeat(2, axis=0)
    b = synth.Batch(pos, sp, cells, np.zeros((2, 3), np.uint8), np.array([0, 0, len(pos)]))
    m = model(cfg, 151)
    v = rng.normal(size=pos.shape)
    hv = _hv(m, b, v)
    ref = om.hessian_vector(om.Model(cfg, synth.model_weights(cfg, 151)), b, v)
    _check(hv, ref, f"isolated atom, correlation {correlation}")
    assert np.all(hv[-1] == 0.0)
    g, posd = _graph(m, b)
    gE = torch.ones(2, dtype=torch.float64, device=device())
    gF = torch.tensor(v, dtype=torch.float32, device=device())
    grad = m.param_grad(g, posd, gE, gF)
    torch.cuda.synchronize()
    assert torch.isfinite(grad).all()


@pytest.mark.parametrize("lmax,C,layers,correlation,n_vec,per_edge", [
    (3, 128, 2, 1, 1, False), (3, 128, 2, 1, 5, False), (3, 64, 2, 1, 2, True), (2, 32, 2, 1, 3, False),
    (2, 32, 1, 1, 3, False), (3, 32, 3, 1, 3, False), (3, 128, 3, 1, 2, False), (2, 64, 2, 2, 4, True)])
def test_batches_of_directions_against_oracle(lmax, C, layers, correlation, n_vec, per_edge):
    # several directions per launch (odd counts leave a workgroup with one),
    # every layer kind and channel count, R per pair and per edge
    import torch
    cfg = synth.ModelConfig(lmax=lmax, channels=C, layers=layers, n_species=3, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0), correlation=correlation)
    rng = np.random.default_rng(160)
    b = synth.concat([synth.jittered_lattice(25, 0.1, 0.3, 3, rng), synth.open_box(17, 3, rng)])
    m = model(cfg, 161)
    m.set_flags(radial_per_edge=per_edge)
    g, pos = _graph(m, b, 0.5)
    V = rng.normal(size=(n_vec,) + b.pos.shape)
    H = m.hessian_vectors(g, pos, torch.tensor(V, dtype=torch.float32, device=device())).cpu().numpy()
    ref = om.Model(cfg, synth.model_weights(cfg, 161))
    for k in range(n_vec):
        _check(H[k].astype(np.float64), om.hessian_vector(ref, b, V[k]), f"direction {k} of {n_vec}")


def test_more_directions_than_one_batch_holds():
    # 270 directions of 90 atoms are more than one batch of atom rows: the
    # first and last direction of each batch against the oracle
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=2, n_species=3, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0))
    b = synth.open_box(90, 3, np.random.default_rng(162))
    m = model(cfg, 163)
    g, pos = _graph(m, b)
    H = m.hessian(g, pos)[0].cpu().numpy().astype(np.float64)
    ref = om.Model(cfg, synth.model_weights(cfg, 163))
    assert np.abs(H - H.T).max() <= REL * np.abs(H).max()
    for k in (0, 182, 183, 269):
        v = np.zeros(270)
        v[k] = 1.0
        _check(H[:, k].reshape(-1, 3), om.hessian_vector(ref, b, v.reshape(-1, 3)), f"column {k}")


def test_directions_in_batches_that_memory_bounds():
    # a direction of this box takes 1.8 GB of tangents, adjoints and messages (16 KB
    # an edge of the middle layer), so two go together; each as if alone
    import torch
    cfg = synth.ModelConfig(lmax=3, channels=128, layers=3, n_species=3, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0))
    b = synth.jittered_lattice(2000, 0.1, 0.3, 3, np.random.default_rng(164))
    m = model(cfg, 165)
    g, pos = _graph(m, b)
    V = torch.tensor(np.random.default_rng(166).normal(size=(3,) + b.pos.shape), dtype=torch.float32, device=device())
    H = m.hessian_vectors(g, pos, V)
    assert m._alloc.bytes_live < 12e9
    for k in range(3):
        one = m.hessian_vector(g, pos, V[k])
        _check(H[k].cpu().numpy().astype(np.float64), one.cpu().numpy().astype(np.float64), f"direction {k}")
