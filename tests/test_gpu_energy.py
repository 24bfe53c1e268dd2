"""GPU energy + forces vs the FP64 oracle (FP32 path).

Tolerances: energy <= 1e-5 relative and forces <= 1e-4 eV/A max-abs against
the FP64 oracle, plus max-abs force error <= 1e-3 of the largest force (the
random-init model has forces of only ~1e-3 eV/A, so the absolute bound alone
would be weak).
"""
import os

import numpy as np
import pytest

import synth
from oracle import model as om
from tests.gpu_util import check_energy, check_forces, gpu_energy_forces, model, say, to_dev

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


def _oracle(cfg, seed_key, b, chunk=None):
    return om.energy_forces(om.Model(cfg, synth.model_weights(cfg, seed_key)), b, edge_chunk=chunk)


@pytest.mark.parametrize("skin", [0.0, 1.0])
def test_tiny_cluster(skin):
    cfg, b = synth.tiny_config()
    say(f"tiny cluster skin={skin}")
    E, F, Ei, _ = gpu_energy_forces(model(cfg, 1), b, skin=skin)
    Er, Fr, Eir = _oracle(cfg, 1, b)
    e = check_energy(E, Er, Eir)
    f = check_forces(F, Fr)
    np.testing.assert_allclose(Ei, Eir, atol=1e-6 * np.abs(Eir).max())
    say(f"  energy rel err {e:.2e}; force err {f[0]:.2e} eV/A ({f[1]:.2e} of max)")


def test_packed_periodic_batch():
    # small periodic boxes (shorter than 2 r_c: several images per pair), l_max 3, 64 channels
    cfg, b, _, _ = synth.differentiation_config(6, 20, 120)
    say(f"packed batch N={b.n_atoms}")
    E, F, Ei, _ = gpu_energy_forces(model(cfg, 3), b, skin=0.5)
    Er, Fr, Eir = _oracle(cfg, 3, b)
    for s in range(b.n_structures):
        a, z = b.offsets[s], b.offsets[s + 1]
        check_energy(E[s:s + 1], Er[s:s + 1], Eir[a:z])
    check_forces(F, Fr)


@pytest.mark.parametrize("unfactorised", [False, True])
def test_single_layer_model(unfactorised):
    # one interaction layer: it is both the first layer (embedding input) and
    # the scalar-output last layer, with its own gate before the readout
    cfg = synth.ModelConfig(lmax=3, channels=32, layers=1, n_species=3, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0))
    b = synth.jittered_lattice(120, 0.1, 0.3, 3, np.random.default_rng(47))
    m = model(cfg, 48)
    if unfactorised:
        m.set_flags(unfactorised_first_layer=True)
    E, F, Ei, _ = gpu_energy_forces(m, b, skin=1.0)
    Er, Fr, Eir = _oracle(cfg, 48, b)
    e = check_energy(E, Er, Eir)
    f = check_forces(F, Fr)
    say(f"single layer (unfactorised {unfactorised}): energy rel err {e:.2e}, force err {f[0]:.2e} eV/A")


def test_three_layer_full_middle_layer():
    # 3 layers: the middle layer runs all 23 paths of l_max 3.
    cfg = synth.ModelConfig(lmax=3, channels=128, layers=3, n_species=4, cutoff=6.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 6.0))
    b = synth.jittered_lattice(150, 0.1, 0.3, 4, np.random.default_rng(41))
    say(f"3-layer N={b.n_atoms}")
    E, F, Ei, _ = gpu_energy_forces(model(cfg, 5), b, skin=1.0)
    Er, Fr, Eir = _oracle(cfg, 5, b, chunk=4096)
    check_energy(E, Er, Eir)
    check_forces(F, Fr)


def test_lmax2_open_cluster_batch():
    cfg = synth.ModelConfig(lmax=2, channels=64, layers=3, n_species=3, cutoff=5.0, avg_neighbors=8.0)
    rng = np.random.default_rng(42)
    b = synth.concat([synth.uniform_cluster(n, 9.0, 1.0, 3, rng) for n in (5, 30, 17)])
    E, F, Ei, _ = gpu_energy_forces(model(cfg, 6), b, skin=0.3)
    Er, Fr, Eir = _oracle(cfg, 6, b)
    for s in range(b.n_structures):
        a, z = b.offsets[s], b.offsets[s + 1]
        check_energy(E[s:s + 1], Er[s:s + 1], Eir[a:z])
    check_forces(F, Fr)


def test_single_structure_3000_atoms_golden():
    path = os.path.join(HERE, "golden", "single_3000.npz")
    ref = np.load(path)
    cfg, b = synth.single_config()
    say("single structure 3000 atoms (stored oracle result)")
    E, F, Ei, g = gpu_energy_forces(model(cfg, 2), b, skin=1.0)
    e = check_energy(E, ref["energy"], ref["atom_energy"])
    f = check_forces(F, ref["forces"])
    np.testing.assert_allclose(Ei, ref["atom_energy"], atol=1e-5 * np.abs(ref["atom_energy"]).max())
    say(f"  energy rel err {e:.2e}; force err {f[0]:.2e} eV/A ({f[1]:.2e} of max)")


def test_net_force_vanishes_and_repeatable():
    import torch
    cfg, b = synth.single_config(n=800)
    m = model(cfg, 2)
    pos, sp = to_dev(b)
    g = m.build_graph(b.offsets, pos, sp, b.cell, b.pbc, cfg.cutoff, 1.0)
    E1, F1, _ = m.energy_forces(g, pos)
    E2, F2, _ = m.energy_forces(g, pos)
    torch.cuda.synchronize()
    assert torch.equal(E1, E2) and torch.equal(F1, F2)
    F = F1.double().cpu().numpy()
    assert np.abs(F.sum(0)).max() < 1e-5 * np.abs(F).max() * np.sqrt(b.n_atoms)


def test_packing_invariance_bitwise():
    # a structure evaluated alone and inside a packed batch gives identical bits
    import torch
    cfg, b, _, _ = synth.differentiation_config(5, 30, 90)
    m = model(cfg, 3)
    E, F, Ei, _ = gpu_energy_forces(m, b, skin=0.5)
    for s in (0, 3):
        one = b.structure(s)
        E1, F1, Ei1, _ = gpu_energy_forces(m, one, skin=0.5)
        a, z = b.offsets[s], b.offsets[s + 1]
        assert E1[0] == E[s]
        assert np.array_equal(F1, F[a:z])
        assert np.array_equal(Ei1, Ei[a:z])


def test_translation_and_image_shift_invariance():
    import torch
    cfg, b, _, _ = synth.differentiation_config(2, 40, 60)
    m = model(cfg, 3)
    E0, F0, _, _ = gpu_energy_forces(m, b, skin=0.5)
    L = b.cell[:, 0, 0]
    owner = np.repeat(np.arange(b.n_structures), np.diff(b.offsets))
    k = np.random.default_rng(5).integers(-2, 3, size=(b.n_atoms, 3))
    moved = synth.Batch(b.pos + k * L[owner][:, None], b.species, b.cell, b.pbc, b.offsets)
    E1, F1, _, _ = gpu_energy_forces(m, moved, skin=0.5)
    np.testing.assert_allclose(E1, E0, rtol=1e-6)
    np.testing.assert_allclose(F1, F0, atol=1e-6 * np.abs(F0).max())


def test_bf16_mode_errors_against_oracle():
    # BF16 operands for the radial-MLP and channel-mix GEMMs (FP32 accumulation);
    # the errors are reported and only bounded loosely.
    ref = np.load(os.path.join(HERE, "golden", "single_3000.npz"))
    cfg, b = synth.single_config()
    E32, F32, _, _ = gpu_energy_forces(model(cfg, 2), b, skin=1.0)
    E16, F16, _, _ = gpu_energy_forces(model(cfg, 2, precision=1), b, skin=1.0)
    fmax = np.abs(ref["forces"]).max()
    e16 = abs(E16[0] - ref["energy"][0]) / abs(ref["energy"][0])
    f16 = np.abs(F16 - ref["forces"]).max() / fmax
    e32 = abs(E32[0] - ref["energy"][0]) / abs(ref["energy"][0])
    f32 = np.abs(F32 - ref["forces"]).max() / fmax
    per_atom = abs(E16[0] - ref["energy"][0]) / b.n_atoms
    say(f"BF16: energy rel err {e16:.2e} ({per_atom:.2e} eV/atom), force err {f16:.2e} of max |F|; "
        f"FP32: {e32:.2e}, {f32:.2e}")
    # rounding the weights to BF16 shifts every atom's energy alike, so the
    # total error grows with N: bound it per atom
    assert per_atom < 1e-3 and f16 < 5e-2
    assert not np.array_equal(F16, F32)


def test_first_layer_factorisation_matches_per_edge_path():
    import torch
    cfg, b = synth.single_config(n=700)
    m = model(cfg, 2)
    E1, F1, Ei1, _ = gpu_energy_forces(m, b, skin=1.0)
    m.set_flags(unfactorised_first_layer=True)
    E2, F2, Ei2, _ = gpu_energy_forces(m, b, skin=1.0)
    assert abs(E1[0] - E2[0]) <= 1e-6 * abs(E2[0])
    assert np.abs(F1 - F2).max() <= 1e-4 * np.abs(F2).max()
    assert not np.array_equal(F1, F2)  # two different evaluation orders


@pytest.mark.parametrize("n_species", [1, 5, 8])
def test_first_layer_factorisation_other_species_counts(n_species):
    # one species (every column of the (component, species) axis kept), an odd
    # count and the largest the factorisation holds in LDS
    cfg = synth.ModelConfig(lmax=3, channels=32, layers=2, n_species=n_species, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0))
    b = synth.jittered_lattice(300, 0.1, 0.3, n_species, np.random.default_rng(130 + n_species))
    m = model(cfg, 131)
    E1, F1, _, _ = gpu_energy_forces(m, b, skin=1.0)
    m.set_flags(unfactorised_first_layer=True)
    E2, F2, _, _ = gpu_energy_forces(m, b, skin=1.0)
    say(f"species {n_species}: |dE| {abs(E1[0] - E2[0]):.1e}, max |dF| {np.abs(F1 - F2).max():.1e}")
    assert abs(E1[0] - E2[0]) <= 1e-6 * abs(E2[0])
    assert np.abs(F1 - F2).max() <= 1e-4 * np.abs(F2).max()
    assert not np.array_equal(F1, F2)


@pytest.mark.parametrize("lmax,channels", [(3, 128), (3, 64), (2, 32)])
def test_fused_last_layer_matches_unfused_path(lmax, channels):
    cfg = synth.ModelConfig(lmax=lmax, channels=channels, layers=2, n_species=4, cutoff=5.0, avg_neighbors=52.36)
    _, b = synth.single_config(n=500)
    m = model(cfg, 5)
    say(f"fused last layer l_max {lmax} C {channels}")
    m.set_flags(fused_last_layer=True)
    E1, F1, Ei1, _ = gpu_energy_forces(m, b, skin=1.0)
    m.set_flags()
    E2, F2, Ei2, _ = gpu_energy_forces(m, b, skin=1.0)
    assert not np.array_equal(F1, F2)  # the two evaluations really differ in order
    assert np.abs(Ei1 - Ei2).max() <= 1e-5 * np.abs(Ei2).max()
    assert abs(E1[0] - E2[0]) <= 1e-6 * abs(E2[0])
    assert np.abs(F1 - F2).max() <= 1e-4 * np.abs(F2).max()


@pytest.mark.parametrize("n,n_species,lmax", [(2, 1, 3), (17, 1, 3), (18, 2, 2), (65, 1, 2), (66, 4, 3), (130, 1, 3)])
def test_first_layer_row_lengths(n, n_species, lmax):
    # every atom inside every other's cutoff: rows of n - 1 edges, at and one
    # past the blocks of 16 edges and tiles of 64 that the first layer takes
    cfg = synth.ModelConfig(lmax=lmax, channels=32, layers=2, n_species=n_species, cutoff=5.0, avg_neighbors=float(n))
    b = synth.uniform_cluster(n, 2.8, 0.3, n_species, np.random.default_rng(170 + n))
    E, F, Ei, g = gpu_energy_forces(model(cfg, 171), b)
    assert g.last_edge_count() == n * (n - 1)
    Er, Fr, Eir = _oracle(cfg, 171, b)
    check_energy(E, Er, Eir)
    check_forces(F, Fr)


@pytest.mark.parametrize("lmax,channels,correlation", [(2, 32, 1), (3, 32, 1), (2, 128, 1), (3, 64, 2), (3, 32, 2)])
@pytest.mark.parametrize("unfactorised", [False, True])
def test_layers_with_every_path(lmax, channels, correlation, unfactorised):
    # rows of 0, 1, 2 and many edges through the kernels of layers with every
    # path and of the scalar-output layer, at every channel count
    cfg = synth.ModelConfig(lmax=lmax, channels=channels, layers=3, n_species=3, cutoff=5.0, avg_neighbors=10.0,
                            correlation=correlation)
    rng = np.random.default_rng(180)
    parts = [synth.uniform_cluster(n, 4.0, 0.9, 3, rng) for n in (1, 2, 3)] + [synth.jittered_lattice(40, 0.1, 0.3, 3, rng)]
    b = synth.concat(parts)
    m = model(cfg, 181)
    if unfactorised:
        m.set_flags(unfactorised_first_layer=True)
    E, F, Ei, _ = gpu_energy_forces(m, b, skin=0.5)
    Er, Fr, Eir = _oracle(cfg, 181, b)
    for s in range(b.n_structures):
        a, z = b.offsets[s], b.offsets[s + 1]
        check_energy(E[s:s + 1], Er[s:s + 1], Eir[a:z])
    check_forces(F, Fr)


@pytest.mark.parametrize("channels,copies,correlation", [(32, 64, 1), (64, 40, 2), (128, 20, 1)])
@pytest.mark.parametrize("bf16", [False, True])
def test_contractions_of_few_and_many_rows(channels, copies, correlation, bf16):
    # the per-atom contractions take another kernel from 1,024 blocks of 32 x 32
    # outputs on: a structure alone is below it in every one, `copies` of it are
    # above it in the mixes (33 atoms: a last row tile of one row), with the same bits
    cfg = synth.ModelConfig(lmax=3, channels=channels, layers=2, n_species=3, cutoff=4.0, avg_neighbors=10.0,
                            correlation=correlation)
    one = synth.jittered_lattice(33, 0.1, 0.3, 3, np.random.default_rng(190))
    b = synth.concat([one] * copies)
    m = model(cfg, 191, precision=int(bf16))
    E1, F1, Ei1, _ = gpu_energy_forces(m, one)
    E, F, Ei, _ = gpu_energy_forces(m, b)
    assert np.array_equal(E, np.repeat(E1, copies))
    assert np.array_equal(F, np.tile(F1, (copies, 1)))
    assert np.array_equal(Ei, np.tile(Ei1, copies))
    if not bf16:
        Er, Fr, Eir = _oracle(cfg, 191, one)
        check_energy(E1, Er, Eir)
        check_forces(F1, Fr)


@pytest.mark.parametrize("flags,launches", [({"unfactorised_first_layer": True}, 0), ({}, 1)])
def test_stages_that_do_not_run_are_not_counted(flags, launches):
    cfg, b = synth.tiny_config()
    m = model(cfg, 1)
    m.set_flags(**flags)
    gpu_energy_forces(m, b)
    m.profile(True)
    gpu_energy_forces(m, b)
    n = m.stage_time("first_fwd")[1]
    m.profile(False)
    assert min(n, 1) == launches


@pytest.mark.parametrize("layers,correlation,flags", [(5, 1, {}), (6, 1, {}), (8, 1, {"unfactorised_first_layer": True}),
                                                      (5, 2, {})])
def test_more_layers_than_a_radial_launch_takes(layers, correlation, flags):
    # the radial rows of all layers go out together, four jobs a launch
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=layers, n_species=3, cutoff=5.0, avg_neighbors=15.0,
                            correlation=correlation)
    b = synth.open_box(24, 3, np.random.default_rng(230))
    m = model(cfg, 231)
    m.set_flags(**flags)
    E, F, Ei, _ = gpu_energy_forces(m, b, skin=0.5)
    Er, Fr, Eir = _oracle(cfg, 231, b)
    check_energy(E, Er, Eir)
    check_forces(F, Fr)


@pytest.mark.parametrize("correlation,scale", [(1, 1e37), (1, 3.4e38), (2, 1e30)])
def test_an_overflow_shows_and_stays_in_its_structure(correlation, scale):
    # one species' embedding near or past what FP32 and BF16 hold: the structure
    # that has it is finite or NaN throughout, the other has the bits it has alone
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=3, n_species=3, cutoff=5.0, avg_neighbors=15.0,
                            correlation=correlation)
    rng = np.random.default_rng(234)
    a, b = synth.open_box(20, 2, rng), synth.open_box(20, 3, rng)
    w = synth.model_weights(cfg, 235)
    flat = synth.flatten_weights(cfg, w)
    flat[2 * cfg.channels:3 * cfg.channels] *= scale
    m = model(cfg, 235)
    m.set_weights(flat)
    E0, F0, _, _ = gpu_energy_forces(m, a)
    E, F, _, _ = gpu_energy_forces(m, synth.concat([a, b]))
    assert np.isfinite(E0).all() and E[0] == E0[0] and np.array_equal(F[:20], F0)
    for x in (E[1:], F[20:]):
        assert np.isfinite(x).all() if scale == 1e37 else np.isnan(x).all()
