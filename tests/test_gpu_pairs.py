"""The radial MLP and its adjoint once per edge pair (the default for layers
whose edges are all in memory at once) against the same model evaluated edge
by edge (E3MI_FLAG_RADIAL_PER_EDGE): an edge and its reverse have exactly
opposite FP64 vectors, so the forward pass (R written to both rows) gives the
same bits, energies included; the adjoint takes the pair's summed dR through
the MLP once, so forces agree to FP32 rounding (max |dF| <= 1e-5 of the
largest force; BF16 mode: 1e-2, one more rounding of the summed dR to BF16).
Cases with several images of one neighbour, an atom that only sees its own
images, open and slab boundaries and a packed batch; each pair-mode result is
also checked against the FP64 oracle."""
import numpy as np
import pytest

import synth
from oracle import model as om
from tests.gpu_util import check_energy, check_forces, gpu_energy_forces, model, record, say

pytestmark = pytest.mark.gpu


def _cases():
    rng = np.random.default_rng(151)
    _, tiny = synth.tiny_config()
    small = synth.jittered_lattice(20, 0.1, 0.3, 4, rng)        # 5.85 A box: several images per pair
    one = synth.Batch(np.array([[0.3, 0.2, 0.1]]), np.zeros(1, np.int32), (np.eye(3) * 2.2)[None],
                      np.ones((1, 3), np.uint8), np.array([0, 1]))   # only its own images
    slab = synth.jittered_lattice(64, 0.1, 0.3, 4, rng)
    slab.pbc = np.array([[1, 1, 0]], np.uint8)
    batch = synth.concat([synth.jittered_lattice(n, 0.1, 0.3, 4, rng) for n in (7, 33, 2)] + [tiny, one])
    return {"tiny_open": tiny, "small_periodic": small, "single_atom_lattice": one, "slab": slab,
            "packed_batch": batch}


CASES = _cases()


def _cfg(lmax, channels, layers):
    return synth.ModelConfig(lmax=lmax, channels=channels, layers=layers, n_species=4, cutoff=5.0,
                             avg_neighbors=synth.nominal_neighbors(0.1, 5.0))


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("arch", [(3, 64, 2), (2, 64, 3)])
def test_pairs_equal_per_edge_and_oracle(name, arch):
    b = CASES[name]
    cfg = _cfg(*arch)
    m = model(cfg, 152)
    m.set_flags(radial_per_edge=True)
    E0, F0, Ei0, _ = gpu_energy_forces(m, b, skin=1.0)
    m.set_flags()
    E1, F1, Ei1, _ = gpu_energy_forces(m, b, skin=1.0)
    fmax = max(np.abs(F0).max(), 1e-30)
    d = float(np.abs(F1 - F0).max())
    say(f"pairs vs per edge ({name}, lmax {arch[0]}, {arch[2]} layers, N={b.n_atoms}): max |dF| {d:.1e}, "
        f"{d / fmax:.1e} of max |F|")
    assert np.array_equal(E0, E1) and np.array_equal(Ei0, Ei1)
    assert d <= 1e-5 * fmax
    Er, Fr, Eir = om.energy_forces(om.Model(cfg, synth.model_weights(cfg, 152)), b)
    check_energy(E1, Er, Eir)
    check_forces(F1, Fr)


@pytest.mark.parametrize("precision,correlation", [(0, 2), (1, 1)])
def test_pairs_larger_box(precision, correlation):
    """400 atoms, 3 layers (a middle layer with every path), the product
    block or the BF16 mode."""
    cfg = synth.ModelConfig(lmax=3, channels=64, layers=3, n_species=4, cutoff=5.0,
                            avg_neighbors=synth.nominal_neighbors(0.1, 5.0), correlation=correlation)
    b = synth.jittered_lattice(400, 0.1, 0.3, 4, np.random.default_rng(153))
    m = model(cfg, 154, precision=precision)
    m.set_flags(radial_per_edge=True)
    E0, F0, Ei0, _ = gpu_energy_forces(m, b, skin=1.0)
    m.set_flags()
    E1, F1, Ei1, _ = gpu_energy_forces(m, b, skin=1.0)
    fmax = np.abs(F0).max()
    d = float(np.abs(F1 - F0).max())
    record("pairs_vs_per_edge", precision=precision, correlation=correlation, max_abs=d, rel_to_max_abs_F=d / fmax)
    assert np.array_equal(E0, E1) and np.array_equal(Ei0, Ei1)
    assert d <= (1e-5 if precision == 0 else 1e-2) * fmax


@pytest.mark.parametrize("n,species_seed", [(1, 5), (4, 6), (5, 7), (16384, 8), (16385, 9)])
def test_selected_edges_and_pairs_at_block_edges(n, species_seed):
    # rows per workgroup (4) and the row count from which the first places of the
    # rows come from scans: the number of selected edges is the oracle's, and every
    # pair has one owner whose radial weights both edges read (energies and forces
    # are those of the edge-by-edge evaluation)
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=2, n_species=2, cutoff=2.5, avg_neighbors=6.5)
    b = synth.jittered_lattice(n, 0.1, 0.3, 2, np.random.default_rng(species_seed))
    m = model(cfg, 196)
    E, F, Ei, g = gpu_energy_forces(m, b, skin=0.3)
    x = b.pos
    L = np.diagonal(np.asarray(b.cell).reshape(-1, 3, 3)[0])
    pbc = np.asarray(b.pbc).reshape(-1, 3)[0]
    if n > 5:
        from scipy.spatial import cKDTree
        tree = cKDTree(np.mod(x, L) if pbc.any() else x, boxsize=L if pbc.any() else None)
        assert g.last_edge_count() == 2 * len(tree.query_pairs(2.5))
    m.set_flags(radial_per_edge=True)
    E1, F1, _, g1 = gpu_energy_forces(m, b, skin=0.3)
    assert g1.last_edge_count() == g.last_edge_count()
    assert abs(E[0] - E1[0]) <= 1e-6 * np.abs(Ei).sum()
    # (a lone atom among its images: forces of rounding alone)
    assert np.abs(F - F1).max() <= 1e-5 * max(np.abs(F1).max(), 1e-2)


@pytest.mark.parametrize("n,species_seed", [(1, 5), (4, 6), (5, 7), (9, 10)])
def test_selected_edges_of_a_few_atoms_and_their_images(n, species_seed):
    # boxes smaller than the cutoff's sphere, counted over the images
    cfg = synth.ModelConfig(lmax=2, channels=32, layers=2, n_species=2, cutoff=2.5, avg_neighbors=6.5)
    b = synth.jittered_lattice(n, 0.1, 0.3, 2, np.random.default_rng(species_seed))
    g = gpu_energy_forces(model(cfg, 196), b, skin=0.3)[3]
    L = np.diagonal(np.asarray(b.cell).reshape(-1, 3, 3)[0])
    shifts = np.stack(np.meshgrid(*[np.arange(-k, k + 1) for k in np.ceil(2.5 / L).astype(int) + 1], indexing="ij"),
                      -1).reshape(-1, 3) * L
    assert np.asarray(b.pbc).all()
    r = np.linalg.norm(b.pos[None, :, None] - b.pos[:, None, None] + shifts, axis=-1)
    assert g.last_edge_count() == int(((r < 2.5) & (r > 0)).sum())
