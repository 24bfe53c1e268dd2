"""Parameter gradients of an energy + force loss (second order through F):
the library's pass behind torch.autograd vs the oracle's double backward.
Bound: relative L2 error of the whole gradient <= 1e-4, and <= 1e-3 per
weight tensor."""
import os

import numpy as np
import pytest

import synth
from oracle import model as om
from tests.gpu_util import check_energy, check_forces, device, gpu_energy_forces, record, say

pytestmark = pytest.mark.gpu


def _gpu_loss_grads(cfg, seed_key, b, e_ref, f_ref, w_e=1.0, w_f=1.0, skin=0.5):
    import torch
    import paper_2605_22698_amd as e3
    d = device()
    wflat = synth.flatten_weights(cfg, synth.model_weights(cfg, seed_key))
    m = e3.Model(cfg.to_json(), wflat, device=d)
    pos = torch.tensor(b.pos, dtype=torch.float64, device=d)
    sp = torch.tensor(b.species, dtype=torch.int32, device=d)
    g = m.build_graph(b.offsets, pos, sp, b.cell, b.pbc, cfg.cutoff, skin)
    w = torch.tensor(wflat, dtype=torch.float64, device=d, requires_grad=True)
    E, F = e3.energy_forces(w, pos, m, g)
    loss = (w_e * torch.mean((E - torch.tensor(e_ref, device=d)) ** 2)
            + w_f * torch.sum((F.double() - torch.tensor(f_ref, device=d)) ** 2) / F.numel())
    loss.backward()
    torch.cuda.synchronize()
    return loss.item(), w.grad.cpu().numpy()


def _compare(cfg, seed_key, b, e_ref, f_ref, w_e=1.0, w_f=1.0, rel=1e-4):
    loss_g, grad_g = _gpu_loss_grads(cfg, seed_key, b, e_ref, f_ref, w_e, w_f)
    m = om.Model(cfg, synth.model_weights(cfg, seed_key))
    loss_o, grads_o = om.loss_and_grads(m, b, e_ref, f_ref, w_e, w_f)
    flat_o = synth.flatten_weights(cfg, grads_o)
    assert abs(loss_g - loss_o) <= 1e-5 * abs(loss_o)
    tot = np.linalg.norm(grad_g - flat_o) / np.linalg.norm(flat_o)
    record("gradient", loss_rel=abs(loss_g - loss_o) / abs(loss_o), grad_rel_l2=float(tot), bound=rel)
    assert tot <= rel
    _per_tensor(cfg, grad_g, flat_o)


def _per_tensor(cfg, grad_g, flat_o):
    off = 0
    for name, shape, _ in synth.weight_shapes(cfg):
        n = int(np.prod(shape))
        a, r = grad_g[off:off + n], flat_o[off:off + n]
        off += n
        nr = np.linalg.norm(r)
        if nr > 1e-9 * np.linalg.norm(flat_o):
            assert np.linalg.norm(a - r) <= 1e-3 * nr, (name, np.linalg.norm(a - r) / nr)
        else:
            assert np.linalg.norm(a) <= 1e-6 * np.linalg.norm(flat_o) + 1e-12, name


def test_energy_and_force_loss_small_batch():
    cfg, b, e_ref, f_ref = synth.differentiation_config(3, 20, 60)
    say(f"grad: batch N={b.n_atoms}")
    _compare(cfg, 3, b, e_ref, f_ref)


def test_force_only_and_energy_only():
    cfg, b, e_ref, f_ref = synth.differentiation_config(2, 25, 40)
    _compare(cfg, 3, b, e_ref, f_ref, w_e=0.0, w_f=1.0)
    _compare(cfg, 3, b, e_ref, f_ref, w_e=1.0, w_f=0.0)


def test_three_layers_lmax2():
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=3, n_species=3, cutoff=5.0, avg_neighbors=20.0)
    rng = np.random.default_rng(61)
    b = synth.concat([synth.jittered_lattice(n, 0.1, 0.3, 3, rng) for n in (18, 33)])
    e_ref = rng.standard_normal(2)
    f_ref = rng.standard_normal((b.n_atoms, 3)) * 0.01
    _compare(cfg, 8, b, e_ref, f_ref)


def test_open_cluster_lmax3_three_layers():
    cfg = synth.ModelConfig(lmax=3, channels=64, layers=3, n_species=3, cutoff=5.0, avg_neighbors=15.0)
    rng = np.random.default_rng(62)
    b = synth.uniform_cluster(20, 8.0, 1.0, 3, rng)
    _compare(cfg, 9, b, rng.standard_normal(1), rng.standard_normal((20, 3)) * 0.01)


@pytest.mark.parametrize("lmax,C,layers", [(2, 32, 2), (3, 64, 3)])
def test_product_block(lmax, C, layers):
    # correlation 2: gradients of w1, w2 and W_lin, and everything upstream of
    # the block through its tangent and reverse
    cfg = synth.ModelConfig(lmax=lmax, channels=C, layers=layers, n_species=4, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0), correlation=2)
    rng = np.random.default_rng(63 + layers)
    b = synth.concat([synth.jittered_lattice(n, 0.1, 0.3, 4, rng) for n in (36, 25)])
    say(f"grad: product block lmax {lmax} C {C} layers {layers} N={b.n_atoms}")
    e_ref = rng.standard_normal(2)
    f_ref = rng.standard_normal((b.n_atoms, 3)) * 0.01
    _compare(cfg, 10, b, e_ref, f_ref)


def test_differentiation_batch_64_structures_golden():
    # the full differentiation batch: 64 periodic boxes of 20-200 atoms, against
    # the oracle's loss and gradient stored by tests/golden/make_golden.py
    import torch
    import paper_2605_22698_amd as e3
    ref = np.load(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "grad_batch_64.npz"))
    cfg, b, e_ref, f_ref = synth.differentiation_config()
    say(f"grad: 64-structure batch N={b.n_atoms}")
    d = device()
    wflat = synth.flatten_weights(cfg, synth.model_weights(cfg, 3))
    m = e3.Model(cfg.to_json(), wflat, device=d)
    pos = torch.tensor(b.pos, dtype=torch.float64, device=d)
    g = m.build_graph(b.offsets, pos, torch.tensor(b.species, dtype=torch.int32, device=d), b.cell, b.pbc,
                      cfg.cutoff, 0.5)
    w = torch.tensor(wflat, dtype=torch.float64, device=d, requires_grad=True)
    E, F = e3.energy_forces(w, pos, m, g)
    loss = (torch.mean((E - torch.tensor(e_ref, device=d)) ** 2)
            + torch.sum((F.double() - torch.tensor(f_ref, device=d)) ** 2) / F.numel())
    loss.backward()
    torch.cuda.synchronize()
    Eh, Fh = E.detach().cpu().numpy(), F.detach().double().cpu().numpy()
    for s in range(b.n_structures):
        a, z = b.offsets[s], b.offsets[s + 1]
        check_energy(Eh[s:s + 1], ref["energy"][s:s + 1], ref["atom_energy"][a:z])
    check_forces(Fh, ref["forces"])
    lo, go = float(ref["loss"]), ref["grad"]
    gg = w.grad.cpu().numpy()
    tot = np.linalg.norm(gg - go) / np.linalg.norm(go)
    record("gradient", loss_rel=abs(loss.item() - lo) / abs(lo), grad_rel_l2=float(tot), bound=1e-4)
    assert abs(loss.item() - lo) <= 1e-5 * abs(lo)
    assert tot <= 1e-4
    _per_tensor(cfg, gg, go)


def test_weights_changed_in_place_and_between_forward_and_backward():
    # a change through .data keeps the tensor's version counter; a second
    # forward with other weights before the first backward must not change
    # what the first backward differentiates
    import torch
    import paper_2605_22698_amd as e3
    cfg, b, e_ref, f_ref = synth.differentiation_config(2, 20, 40)
    d = device()
    w0 = synth.flatten_weights(cfg, synth.model_weights(cfg, 3))
    w1 = synth.flatten_weights(cfg, synth.model_weights(cfg, 4))
    m = e3.Model(cfg.to_json(), w0, device=d)
    pos = torch.tensor(b.pos, dtype=torch.float64, device=d)
    g = m.build_graph(b.offsets, pos, torch.tensor(b.species, dtype=torch.int32, device=d), b.cell, b.pbc,
                      cfg.cutoff, 0.5)

    def loss_of(E, F):
        return (torch.mean((E - torch.tensor(e_ref, device=d)) ** 2)
                + torch.sum((F.double() - torch.tensor(f_ref, device=d)) ** 2) / F.numel())

    def reference(wv):
        mm = e3.Model(cfg.to_json(), wv, device=d)
        ww = torch.tensor(wv, dtype=torch.float64, device=d, requires_grad=True)
        gg = mm.build_graph(b.offsets, pos, torch.tensor(b.species, dtype=torch.int32, device=d), b.cell, b.pbc,
                            cfg.cutoff, 0.5)
        E, F = e3.energy_forces(ww, pos, mm, gg)
        loss_of(E, F).backward()
        return E.detach().cpu().numpy(), ww.grad.cpu().numpy()

    E_ref0, G_ref0 = reference(w0)
    E_ref1, G_ref1 = reference(w1)
    w = torch.tensor(w0, dtype=torch.float64, device=d, requires_grad=True)
    E, F = e3.energy_forces(w, pos, m, g)
    assert np.array_equal(E.detach().cpu().numpy(), E_ref0)
    w.data.copy_(torch.tensor(w1, device=d))          # in place, version counter unchanged
    E, F = e3.energy_forces(w, pos, m, g)
    assert np.array_equal(E.detach().cpu().numpy(), E_ref1)
    # two forwards, then the first one's backward
    wa = torch.tensor(w0, dtype=torch.float64, device=d, requires_grad=True)
    wb = torch.tensor(w1, dtype=torch.float64, device=d, requires_grad=True)
    Ea, Fa = e3.energy_forces(wa, pos, m, g)
    Eb, Fb = e3.energy_forces(wb, pos, m, g)
    loss_of(Ea, Fa).backward()
    loss_of(Eb, Fb).backward()
    torch.cuda.synchronize()
    assert np.array_equal(wa.grad.cpu().numpy(), G_ref0)
    assert np.array_equal(wb.grad.cpu().numpy(), G_ref1)


@pytest.mark.parametrize("lmax,C,layers,correlation,per_edge", [
    (3, 32, 1, 1, False), (3, 128, 2, 1, True), (2, 64, 2, 1, False), (3, 64, 3, 1, True), (3, 32, 2, 2, False)])
def test_gradient_of_every_layer_kind(lmax, C, layers, correlation, per_edge):
    # every layer kind and channel count, the radial MLP per edge pair and per
    # edge, atom counts at and past the 64 that the species sums take at once
    import torch
    import paper_2605_22698_amd as e3
    cfg = synth.ModelConfig(lmax=lmax, channels=C, layers=layers, n_species=3, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0), correlation=correlation)
    rng = np.random.default_rng(190)
    b = synth.concat([synth.jittered_lattice(40, 0.1, 0.3, 3, rng), synth.open_box(24 + (C == 64), 3, rng)])
    w = synth.model_weights(cfg, 191)
    d = device()
    m = e3.Model(cfg.to_json(), synth.flatten_weights(cfg, w), device=d)
    m.set_flags(radial_per_edge=per_edge)
    pos = torch.tensor(b.pos, dtype=torch.float64, device=d)
    g = m.build_graph(b.offsets, pos, torch.tensor(b.species, dtype=torch.int32, device=d), b.cell, b.pbc, cfg.cutoff, 0.5)
    e_ref, f_ref = rng.standard_normal(2), rng.standard_normal(b.pos.shape)
    E, F, _ = m.energy_forces(g, pos)
    gE = E - torch.tensor(e_ref, device=d)  # d/dE of mean_s (E - E*)^2, S = 2
    gF = 2 * (F.double() - torch.tensor(f_ref, device=d)) / F.numel()
    grad = m.param_grad(g, pos, gE, gF).cpu().numpy()
    _, grads_o = om.loss_and_grads(om.Model(cfg, w), b, e_ref, f_ref)
    flat_o = synth.flatten_weights(cfg, grads_o)
    assert np.linalg.norm(grad - flat_o) <= 1e-4 * np.linalg.norm(flat_o)
    _per_tensor(cfg, grad, flat_o)


@pytest.mark.parametrize("precision", [0, 1])
def test_weights_replaced_from_the_device(precision):
    # a device tensor gives the bits of the host vector; a value that is not
    # finite is refused and leaves the weights alone
    import torch
    import paper_2605_22698_amd as e3
    cfg, b, _, _ = synth.differentiation_config(2, 20, 30)
    d = device()
    w0, w1 = (synth.flatten_weights(cfg, synth.model_weights(cfg, k)) for k in (200, 201))
    fresh = e3.Model(cfg.to_json(), w1, precision=precision, device=d)
    m = e3.Model(cfg.to_json(), w0, precision=precision, device=d)
    pos = torch.tensor(b.pos, dtype=torch.float64, device=d)
    sp = torch.tensor(b.species, dtype=torch.int32, device=d)

    def evaluate(x):
        E, F, _ = x.energy_forces(x.build_graph(b.offsets, pos, sp, b.cell, b.pbc, cfg.cutoff), pos)
        return E.cpu().numpy(), F.cpu().numpy()
    ref = evaluate(fresh)
    for w in (torch.tensor(w1, device=d), torch.tensor(w1), w1):
        m.set_weights(w0)
        m.set_weights(w)
        assert all(np.array_equal(a, r) for a, r in zip(evaluate(m), ref))
    for at in (0, w0.size - 1):
        bad = torch.tensor(w0, device=d)
        bad[at] = float("nan")
        with pytest.raises(e3.E3miError, match="not finite"):
            m.set_weights(bad)
        assert all(np.array_equal(a, r) for a, r in zip(evaluate(m), ref))


@pytest.mark.parametrize("precision", [0, 1])
def test_weights_rounded_to_fp32_first(precision):
    # weights that FP32 cannot hold, next to halfway between BF16 neighbours:
    # rounded to FP32 first (to the tie) they give what FP32 weights give, bit for bit
    import paper_2605_22698_amd as e3
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=2, n_species=2, cutoff=4.0, avg_neighbors=8.0)
    b = synth.uniform_cluster(20, 3.0, 0.9, 2, np.random.default_rng(140))
    w = synth.flatten_weights(cfg, synth.model_weights(cfg, 141)).astype(np.float32)
    tie = ((w.view(np.uint32) & 0xffff0000) | 0x8000).view(np.float32).astype(np.float64)
    near = tie * (1.0 + 2.0 ** -40)
    assert np.array_equal(near.astype(np.float32).astype(np.float64), tie) and not np.array_equal(near, tie)
    out = []
    for v in (tie, near):
        m = e3.Model(cfg.to_json(), v, precision=precision, device=device())
        m.set_flags(unfactorised_first_layer=True)  # the factorisation forms products in FP64
        out.append(gpu_energy_forces(m, b)[:3])
    for x, y in zip(*out):
        assert np.array_equal(x, y)


def test_weights_replaced_while_another_device_is_current():
    # from a host vector and from either device's memory
    import torch
    import paper_2605_22698_amd as e3
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    cfg, b, _, _ = synth.differentiation_config(2, 20, 30)
    w0, w1 = (synth.flatten_weights(cfg, synth.model_weights(cfg, k)) for k in (200, 201))
    d = torch.device("cuda:1")
    pos = torch.tensor(b.pos, dtype=torch.float64, device=d)
    sp = torch.tensor(b.species, dtype=torch.int32, device=d)

    def evaluate(x):
        with torch.cuda.device(d):
            E, F, _ = x.energy_forces(x.build_graph(b.offsets, pos, sp, b.cell, b.pbc, cfg.cutoff), pos)
            return E.cpu().numpy(), F.cpu().numpy()
    ref = evaluate(e3.Model(cfg.to_json(), w1, device=d))
    for w in (w1, torch.tensor(w1, device=d), torch.tensor(w1, device="cuda:0")):
        m = e3.Model(cfg.to_json(), w0, device=d)
        with torch.cuda.device(0):
            m.set_weights(w)
        assert all(np.array_equal(a, r) for a, r in zip(evaluate(m), ref))


def test_weights_of_a_model_on_the_default_device_stay_on_the_device(monkeypatch):
    # the default device has no index, tensors' devices have one: the library is
    # handed the tensor's own memory, in set_weights and under autograd
    import torch
    import paper_2605_22698_amd as e3
    cfg, b, _, _ = synth.differentiation_config(2, 20, 30)
    w0, w1 = (synth.flatten_weights(cfg, synth.model_weights(cfg, k)) for k in (200, 201))
    m = e3.Model(cfg.to_json(), w0)
    pos = torch.tensor(b.pos, dtype=torch.float64, device="cuda")
    sp = torch.tensor(b.species, dtype=torch.int32, device="cuda")
    g = m.build_graph(b.offsets, pos, sp, b.cell, b.pbc, cfg.cutoff)
    given = []
    real = e3.lib()

    class Spy:
        def __getattr__(self, name):
            if name == "e3mi_model_set_weights":
                given.append(name)
                return lambda handle, p, n: (given.__setitem__(-1, p), real.e3mi_model_set_weights(handle, p, n))[1]
            return getattr(real, name)
    monkeypatch.setattr(e3, "lib", Spy)
    w = torch.tensor(w1, device="cuda", requires_grad=True)
    m.set_weights(w)
    E, _ = e3.energy_forces(w, pos, m, g)
    E.sum().backward()
    assert set(given) == {w.data_ptr()}
    assert m.device == torch.device("cuda")


@pytest.mark.parametrize("channels,copies", [(128, (6, 6, 7))])
def test_gradient_of_many_copies_of_a_cell(channels, copies):
    # n copies of a periodic cell have n times its gradient, sums of the same
    # rows over and over: what differs is the rounding of long FP32 sums. The
    # middle layer's widest tensors are sums over 180,000 pairs. A sum in FP32
    # over at most 1,024 rows takes 128 additions on the matrix cores (two
    # terms, 16 rows at a time), each off by half of 2^-24 of it or so either way,
    # so about sqrt(128) of them add up (the widest tensor's sums are twice as
    # long, as many as there is room for)
    import torch
    import paper_2605_22698_amd as e3
    cfg = synth.ModelConfig(lmax=3, channels=channels, layers=3, n_species=3, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0))
    rng = np.random.default_rng(220)
    cell = synth.jittered_lattice(27, 0.1, 0.3, 3, rng)
    v = 0.1 * rng.standard_normal(cell.pos.shape)
    d = device()
    m = e3.Model(cfg.to_json(), synth.flatten_weights(cfg, synth.model_weights(cfg, 221)), device=d)

    def gradient(k):
        n = int(np.prod(k))
        at = np.stack(np.meshgrid(*[np.arange(x) for x in k], indexing="ij"), -1).reshape(-1, 1, 3)
        pos = torch.tensor((cell.pos[None] + at * np.diagonal(cell.cell[0])).reshape(-1, 3), device=d)
        sp = torch.tensor(np.tile(cell.species, n), dtype=torch.int32, device=d)
        g = m.build_graph(np.array([0, 27 * n]), pos, sp, cell.cell * np.array(k)[None, :, None], cell.pbc, cfg.cutoff, 0.1)
        gE = torch.ones(1, dtype=torch.float64, device=d)
        return m.param_grad(g, pos, gE, torch.tensor(np.tile(v, (n, 1)), device=d)).cpu().numpy() / n
    one, many = gradient((1, 1, 1)), gradient(copies)
    off, worst = 0, {}
    for name, shape, _ in synth.weight_shapes(cfg):
        n = int(np.prod(shape))
        a, r = many[off:off + n], one[off:off + n]
        off += n
        if np.linalg.norm(r) > 1e-9 * np.linalg.norm(one):
            worst[name] = float(np.linalg.norm(a - r) / np.linalg.norm(r))
    bound = np.sqrt(128) * 2.0 ** -25
    record("gradient_of_copies", rel_l2={k: f"{x:.1e}" for k, x in worst.items()}, bound=bound)
    assert max(worst.values()) <= bound, worst


@pytest.mark.parametrize("layers", [5, 6])
def test_gradient_of_many_layers(layers):
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=layers, n_species=3, cutoff=5.0, avg_neighbors=15.0)
    rng = np.random.default_rng(232)
    b = synth.open_box(24, 3, rng)
    _compare(cfg, 233, b, rng.standard_normal(1), rng.standard_normal((24, 3)) * 0.01)
