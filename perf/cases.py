"""The work that users of this library have it do, as cases to be timed.

listed() and draw() name the cases, prepare() makes what a user's program holds
before the call, run() is one pass through the public entry points, work() the
bytes and operations of a pass that no implementation can do without, exact()
what the pass returns, evaluated in 64 bits with plain torch.

A case:
  kind         what a pass is
                 "energy"   energy + forces on a neighbour list that is held (a
                            calculator called with new positions)
                 "fresh"    neighbour lists built and energy + forces taken of
                            structures that were not seen before (screening)
                 "md"       `steps` steps of velocity-Verlet MD, then the frame
                 "train"    energies and forces, a loss on both, its gradient
                            with respect to the weights, a step of SGD
                 "hessian"  the full Hessian of every structure
                 "hvp"      `vectors` Hessian-vector products
  structures   how many, with lo..hi atoms, spread evenly between the two
  open         every axis open, else every axis periodic
  and the model: lmax, channels, layers, species, cutoff, correlation (2: with
  the product block), coulomb, bf16 (the mixed mode, else FP32)

Structures are liquid-like: sites of a cubic lattice at 0.1 atoms/A^3 with
Gaussian jitter. Weights are Gaussian with the spread 1/sqrt(fan-in) that keeps
every layer's activations near one. The species' reference energies are of the
size of isolated atoms' total energies, as trained models carry them.
"""
import itertools
import json
import math

import numpy as np
import torch
import torch.utils.checkpoint

import paper_2605_22698_amd as e3

DENSITY = 0.1            # atoms / A^3
HIDDEN, BASIS, READOUT, ENVELOPE = 64, 8, 16, 6
SOFT_CORE = 2.0          # A
K_E = 14.399645478425668  # eV A
ACCEL = 0.009648533      # A/fs^2 per (eV/A)/amu
KB = 8.617333262e-5      # eV/K
MASSES = (1.008, 12.011, 14.007, 15.999, 32.06)
ATOM_ENERGY = (-13.6, -1029.7, -1485.3, -2042.6, -10832.3)  # eV
DT = 0.5                 # fs
SKIN, REBUILD = 1.0, 20
RATE = 1e-7              # SGD


def _case(name, kind, structures, lo, hi, **more):
    c = {"kind": kind, "structures": structures, "lo": lo, "hi": hi, "open": False, "lmax": 3, "channels": 128,
         "layers": 2, "species": 4, "cutoff": 5.0, "correlation": 1, "coulomb": False, "bf16": False, "steps": 0,
         "vectors": 0}
    c.update(more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small molecule in a relaxation or a path search: one call at a time, so latency and launches
        _case("energy_24_small_model", "energy", 1, 24, 24, open=True, lmax=2, channels=32, species=3),
        # a peptide of 138 atoms in the gas phase
        _case("energy_138_open", "energy", 1, 138, 138, open=True),
        # a small protein in the gas phase, MD
        _case("md_1205_open", "md", 1, 1205, 1205, open=True, steps=20),
        # the headline workload: MD of a periodic box
        _case("md_3000", "md", 1, 3000, 3000, steps=20),
        # the same box in the mixed mode
        _case("energy_3000_bf16", "energy", 1, 3000, 3000, bf16=True),
        # screening: a batch of molecules, each seen once
        _case("fresh_64_molecules", "fresh", 64, 10, 31, open=True),
        # charged clusters with long-range electrostatics
        _case("energy_64_charged", "energy", 64, 20, 200, open=True, coulomb=True),
        # the model with the product block
        _case("energy_3000_product", "energy", 1, 3000, 3000, correlation=2),
        # a large box with a deeper model and a longer cutoff: layers that carry every path
        _case("energy_20000_deep", "energy", 1, 20000, 20000, layers=3, cutoff=6.0),
        # training on energies and forces
        _case("train_64_boxes", "train", 64, 20, 200, channels=64, species=5),
        # vibrational analysis: full Hessians of a batch of molecules
        _case("hessian_64_molecules", "hessian", 64, 10, 31, open=True),
        # an iterative eigensolver on a box: one product at a time
        _case("hvp_3000", "hvp", 1, 3000, 3000, vectors=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("energy", "energy", "fresh", "md", "train", "hessian", "hvp"))
    m = {"lmax": rng.choice((2, 3, 3)), "channels": rng.choice((32, 64, 128, 128)), "layers": rng.choice((2, 2, 3)),
         "species": rng.randint(2, 5), "cutoff": round(rng.uniform(4.5, 6.0), 2), "open": rng.random() < 0.5,
         "correlation": rng.choice((1, 1, 1, 2))}
    # models whose layers carry every path between all orders take several times the work per edge
    heavy = m["layers"] > 2 or m["correlation"] == 2
    if kind == "energy":
        one = rng.random() < 0.5
        n = _log(rng, 20, 4000) if one else _log(rng, 20, 200)
        m["bf16"] = rng.random() < 0.3
        if m["open"] and rng.random() < 0.4:
            m.update(coulomb=True, correlation=1)
        return _case(None, kind, 1 if one else rng.randint(2, 32), n if one else max(10, n // 4), n, **m)
    if kind == "fresh":
        n = _log(rng, 12, 200)
        return _case(None, kind, rng.randint(4, 96), max(8, n // 3), n, **m)
    if kind == "md":
        n = _log(rng, 60, 600 if heavy else 3500)
        m["bf16"] = rng.random() < 0.3
        return _case(None, kind, 1, n, n, steps=rng.choice((10, 20)), **m)
    if kind == "train":
        n = _log(rng, 20, 200)
        return _case(None, kind, rng.randint(2, 8 if heavy else 48), max(10, n // 4), n, **dict(m, channels=rng.choice((32, 64))))
    if kind == "hessian":
        n = rng.randint(9, 16 if heavy else 31)
        return _case(None, kind, rng.randint(1, 16 if heavy else 56), max(6, n // 3), n, **dict(m, open=True))
    n = _log(rng, 60, 300 if heavy else 2500)
    return _case(None, kind, 1, n, n, vectors=rng.randint(1, 6), **m)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _sizes(case):
    s, lo, hi = case["structures"], case["lo"], case["hi"]
    return [lo + int((hi - lo + 1) * ((k * 0.6180339887498949) % 1.0)) if s > 1 else hi for k in range(s)]


def _neighbours(cutoff):
    return DENSITY * 4.0 / 3.0 * math.pi * cutoff ** 3


def _inputs(case, seed):
    """(pos [N, 3], species [N], cell [S, 3, 3], pbc [S, 3], offsets [S+1], rng), on the host."""
    rng = np.random.default_rng([int(seed), 11])
    pos, cell = [], []
    for n in _sizes(case):
        side = (n / DENSITY) ** (1.0 / 3.0)
        m = int(math.ceil(round(n ** (1.0 / 3.0), 9)))
        site = np.sort(rng.choice(m ** 3, size=n, replace=False))
        at = np.stack([site // (m * m), (site // m) % m, site % m], 1) + 0.5
        x = at * (side / m) + rng.normal(0.0, 0.3, (n, 3))
        pos.append(x if case["open"] else x - np.floor(x / side) * side)
        cell.append(np.eye(3) * side)
    offsets = np.concatenate([[0], np.cumsum(_sizes(case))]).astype(np.int64)
    species = rng.integers(0, case["species"], offsets[-1]).astype(np.int32)
    pbc = np.full((case["structures"], 3), 0 if case["open"] else 1, np.uint8)
    return np.concatenate(pos), species, np.stack(cell), pbc, offsets, rng


def _paths(case, t):
    lin = [0] if t == 1 else range(case["lmax"] + 1)
    ls = range(case["lmax"] + 1)
    return [(a, b, c) for c in ls for a in lin for b in ls if abs(a - b) <= c <= a + b and (a + b + c) % 2 == 0]


def _pairs(case, top):
    ls = range(case["lmax"] + 1)
    return [(a, b, c) for c in range(top + 1) for a in ls for b in ls if a <= b and abs(a - b) <= c <= a + b and (a + b + c) % 2 == 0]


def _top(case, t):
    return 0 if t == case["layers"] else case["lmax"]


def _shapes(case):
    """(name, shape, fan-in) of the weight tensors in the order of the weight vector."""
    c, ns = case["channels"], case["species"]
    out = [("emb", (ns, c), ns)]
    for t in range(1, case["layers"] + 1):
        ps = _paths(case, t)
        out += [("rad1_%d" % t, (BASIS, HIDDEN), BASIS), ("rad2_%d" % t, (HIDDEN, HIDDEN), HIDDEN), ("rad3_%d" % t, (HIDDEN, len(ps) * c), HIDDEN)]
        for l in range(case["lmax"] + 1):
            n = sum(p[2] == l for p in ps) * c
            out.append(("mix_%d_%d" % (t, l), (n, c), n))
        out += [("self_%d_%d" % (t, l), (c, c), c) for l in ([0] if t == 1 else range(case["lmax"] + 1))]
        if case["correlation"] == 2:
            n = len(_pairs(case, _top(case, t)))
            out += [("sym1_%d" % t, (ns, _top(case, t) + 1, c), 2), ("sym2_%d" % t, (ns, n, c), n)]
            out += [("lin_%d_%d" % (t, l), (c, c), c) for l in range(_top(case, t) + 1)]
    out += [("read1", (c, READOUT), c), ("read2", (READOUT, 1), READOUT), ("e0", (ns,), 0)]
    if case["coulomb"]:
        out += [("qhead", (c,), 10 * c), ("qbias", (ns,), 10 * ns)]  # charges of a few tenths of e
    return out


def _weights(case, seed):
    rng = np.random.default_rng([int(seed), 12])
    parts = [rng.standard_normal(math.prod(s)) / math.sqrt(f) if f else np.array(ATOM_ENERGY[:s[0]]) for _, s, f in _shapes(case)]
    return np.concatenate(parts).astype(np.float32).astype(np.float64)  # trained in 32 bits


def _config(case):
    return {"lmax": case["lmax"], "channels": case["channels"], "layers": case["layers"], "n_species": case["species"],
            "cutoff": case["cutoff"], "avg_neighbors": _neighbours(case["cutoff"]), "n_basis": BASIS, "envelope_p": ENVELOPE,
            "radial_hidden": HIDDEN, "readout_hidden": READOUT, "correlation": case["correlation"], "coulomb": case["coulomb"],
            "soft_core_r0": SOFT_CORE}


def _targets(case, species, offsets, rng):
    e0 = np.array(ATOM_ENERGY).astype(np.float32).astype(np.float64)[species]
    return np.add.reduceat(e0, offsets[:-1]) + rng.standard_normal(len(offsets) - 1), rng.standard_normal((len(species), 3))


def _velocities(species, rng):
    m = np.array(MASSES)[species]
    v = rng.standard_normal((len(species), 3)) * np.sqrt(KB * 300.0 * ACCEL / m)[:, None]
    return v - (m[:, None] * v).sum(0) / m.sum()


def _charges(case, rng):
    return rng.integers(-1, 2, case["structures"]).astype(np.float64)


def prepare(case, seed):
    dev = torch.device("cuda")
    pos, species, cell, pbc, offsets, rng = _inputs(case, seed)
    w = _weights(case, seed)
    model = e3.Model(json.dumps(_config(case)), w, e3.BF16_MIX if case["bf16"] else e3.FP32, device=dev)
    s = {"kind": case["kind"], "model": model, "pos": torch.tensor(pos, device=dev), "species": torch.tensor(species, device=dev),
         "offsets": offsets, "cell": cell, "pbc": pbc, "cutoff": case["cutoff"]}
    if case["kind"] == "md":
        s["md"] = e3.MD(model, offsets, s["pos"], torch.tensor(_velocities(species, rng), device=dev), s["species"],
                        np.array(MASSES[:case["species"]]), cell, pbc, case["cutoff"], SKIN, REBUILD)
        s["steps"] = case["steps"]
        s["energy"] = torch.empty(1, dtype=torch.float64, device=dev)
    elif case["kind"] != "fresh":
        s["graph"] = model.build_graph(offsets, s["pos"], s["species"], cell, pbc, case["cutoff"], SKIN)
    if case["coulomb"]:
        s["graph"].set_total_charge(_charges(case, rng))
    if case["kind"] == "train":
        e, f = _targets(case, species, offsets, rng)
        s.update(e_ref=torch.tensor(e, device=dev), f_ref=torch.tensor(f, dtype=torch.float32, device=dev),
                 weights=torch.tensor(w, dtype=torch.float32, device=dev, requires_grad=True), heads=case["species"])
    if case["kind"] == "hvp":
        s["v"] = torch.tensor(rng.standard_normal((case["vectors"], len(pos), 3)), dtype=torch.float32, device=dev)
    return s


def run(s):
    model, pos = s["model"], s["pos"]
    if s["kind"] == "energy":
        e, f, _ = model.energy_forces(s["graph"], pos)
        return {"energy": e, "forces": f}
    if s["kind"] == "fresh":
        graph = model.build_graph(s["offsets"], pos, s["species"], s["cell"], s["pbc"], s["cutoff"])
        e, f, _ = model.energy_forces(graph, pos)
        return {"energy": e, "forces": f}
    if s["kind"] == "md":
        s["md"].step(s["steps"], DT, s["energy"])
        x, v, f = s["md"].state()
        return {"energy": s["energy"], "positions": x, "velocities": v.float(), "forces": f}  # a frame as it is stored
    if s["kind"] == "train":
        w = s["weights"]
        e, f = e3.energy_forces(w, pos, model, s["graph"])
        loss = (e - s["e_ref"]).square().mean() + (f - s["f_ref"]).square().mean()
        (grad,) = torch.autograd.grad(loss, w)
        with torch.no_grad():
            w -= RATE * grad
        n = s["heads"]  # the reference energies' gradient is by far the largest
        return {"energy": e.detach(), "forces": f.detach(), "grad": grad[:-n], "grad_e0": grad[-n:], "weights": w.detach()}
    if s["kind"] == "hessian":
        return model.hessian(s["graph"], pos)
    return model.hessian_vectors(s["graph"], pos, s["v"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _edges_of(case):
    """Expected directed edges inside the cutoff."""
    rc, total = case["cutoff"], 0.0
    for n in _sizes(case):
        if not case["open"]:
            total += n * _neighbours(rc)
            continue
        side = (n / DENSITY) ** (1.0 / 3.0)
        g = (np.arange(24) + 0.5) / 12.0 * rc - rc  # differences of two points of the cube, |d| < rc
        d = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
        d = d[(d * d).sum(1) < rc * rc]
        total += n * (n - 1) / side ** 3 * np.maximum(0.0, 1.0 - np.abs(d) / side).prod(1).sum() * (rc / 12.0) ** 3
    return total


def work(case):
    """Flops: the radial MLP once per pair of an edge and its reverse, the tensor product per edge, the mixes per atom;
    the first layer with its sum taken per sender species before its output layer; only the orders that reach the energy.
    An adjoint with respect to the positions costs what the forward pass does in the MLPs and mixes and twice that in the
    tensor product; a tangent pass the same as the forward pass again, and its reverse twice. Bytes: the arguments and
    results, and the list of edges (sender and image) once."""
    n, edges = sum(_sizes(case)), _edges_of(case)
    c, nc = case["channels"], (case["lmax"] + 1) ** 2
    weights = sum(math.prod(s) for _, s, _ in _shapes(case))
    mlp = tensor = 0.0
    for t in range(1, case["layers"] + 1):
        last = t == case["layers"] and case["correlation"] == 1
        paths = [p for p in _paths(case, t) if not last or p[2] == 0]
        comps = 1 if last else nc
        mlp += edges / 2 * 2.0 * (BASIS * HIDDEN + HIDDEN * HIDDEN)
        if t == 1:
            tensor += edges * 2.0 * HIDDEN * comps
            mlp += n * 2.0 * comps * c * case["species"] * HIDDEN
        else:
            mlp += edges / 2 * 2.0 * HIDDEN * len(paths) * c
            tensor += edges * 2.0 * c * sum((2 * a + 1) * (2 * o + 1) for a, _, o in paths)
            mlp += n * 2.0 * c * c * sum(2 * o + 1 for _, _, o in paths)
        mlp += n * 2.0 * c * c * (1 if t == 1 else comps)
        if case["correlation"] == 2:
            mlp += n * c * 6.0 * sum((2 * a + 1) * (2 * b + 1) for a, b, _ in _pairs(case, _top(case, t)))
            mlp += n * 2.0 * c * c * (_top(case, t) + 1) ** 2
    ef = 2 * mlp + 3 * tensor + (20.0 * sum(k * k for k in _sizes(case)) if case["coulomb"] else 0.0)
    passes = max(1, case["steps"])
    flops, moved = passes * ef, 36.0 * n + 8.0 * edges + 4.0 * weights
    if case["kind"] == "md":
        moved = passes * (84.0 * n + 8.0 * edges) + 4.0 * weights
    if case["kind"] == "train":
        flops, moved = ef + 4 * mlp + 5 * tensor, 48.0 * n + 8.0 * edges + 12.0 * weights
    if case["kind"] in ("hessian", "hvp"):
        k = case["vectors"] or 3 * max(_sizes(case))
        share = 1.0 if case["vectors"] else n / (max(_sizes(case)) * case["structures"])  # a product covers the structures that have the atom
        flops = mlp + tensor + k * share * (3 * mlp + 5 * tensor)
        moved = 28.0 * n + 8.0 * edges + 4.0 * weights + (24.0 * n * k if case["vectors"] else 36.0 * sum(v * v for v in _sizes(case)))
    return {"bytes": moved, "flops": flops}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _harmonics(d, lmax):
    """Real harmonics of the directions of d [E, 3], sum of squares 2l + 1 for each l."""
    x, y, z = (d / d.norm(dim=-1, keepdim=True)).unbind(-1)
    q = math.sqrt
    out = [torch.ones_like(x), q(3) * y, q(3) * z, q(3) * x]
    out += [q(15) * x * y, q(15) * y * z, q(5) / 2 * (3 * z * z - 1), q(15) * x * z, q(15) / 2 * (x * x - y * y)]
    if lmax > 2:
        out += [q(35 / 8) * y * (3 * x * x - y * y), q(105) * x * y * z, q(21 / 8) * y * (5 * z * z - 1), q(7) / 2 * z * (5 * z * z - 3),
                q(21 / 8) * x * (5 * z * z - 1), q(105) / 2 * z * (x * x - y * y), q(35 / 8) * x * (x * x - 3 * y * y)]
    return torch.stack(out, -1)


def _couplings():
    """(l1, l2, l3) -> [2l1+1, 2l2+1, 2l3+1]: integrals of three harmonics over the sphere (exact quadrature), with unit columns."""
    u, wu = np.polynomial.legendre.leggauss(8)
    f = np.arange(16) * (2 * math.pi / 16)
    s = np.sqrt(1 - u * u)
    pts = np.stack([s[:, None] * np.cos(f), s[:, None] * np.sin(f), np.repeat(u[:, None], 16, 1)], -1).reshape(-1, 3)
    y, wt = _harmonics(torch.tensor(pts), 3), torch.tensor(np.repeat(wu, 16) / 32.0)
    out = {}
    for a, b, c in itertools.product(range(4), repeat=3):
        if abs(a - b) <= c <= a + b and (a + b + c) % 2 == 0:
            g = torch.einsum("n,ni,nj,nk->ijk", wt, *(y[:, l * l:(l + 1) ** 2] for l in (a, b, c)))
            out[a, b, c] = g / g[:, :, :1].norm()
    return out


def _edge_list(pos, cell, offsets, is_open, cutoff):
    """(receiver, sender, image displacement) of every directed edge inside the cutoff, by comparing all pairs."""
    dst, src, sh = [], [], []
    for s in range(len(offsets) - 1):
        a, b = int(offsets[s]), int(offsets[s + 1])
        x, side = pos[a:b], float(cell[s, 0, 0])
        k = 0 if is_open else int(math.ceil(cutoff / side))
        for image in itertools.product(range(-k, k + 1), repeat=3):
            t = torch.tensor(image, dtype=pos.dtype, device=pos.device) * side
            rows = max(1, 20_000_000 // (b - a))
            for r in range(0, b - a, rows):
                d = x[None] - x[r:r + rows, None] + t
                near = d.square().sum(-1) < cutoff * cutoff
                if not any(image):
                    near[torch.arange(near.shape[0]), torch.arange(r, r + near.shape[0])] = False
                i, j = near.nonzero(as_tuple=True)
                dst.append(i + a + r)
                src.append(j + a)
                sh.append(t.expand(len(i), 3))
    return torch.cat(dst), torch.cat(src), torch.cat(sh)


class _Exact:
    """The model in 64 bits: atom energies as a differentiable function of positions and weights."""

    def __init__(self, case, flat, species, offsets):
        self.case, self.offsets = case, offsets
        self.dev = flat.device
        self.species = torch.tensor(species.astype(np.int64), device=self.dev)
        self.owner = torch.tensor(np.repeat(np.arange(len(offsets) - 1), np.diff(offsets)), device=self.dev)
        self.cg = {k: v.to(self.dev) for k, v in _couplings().items()}
        self.w, at = {}, 0
        for name, shape, _ in _shapes(case):
            self.w[name] = flat[at:at + math.prod(shape)].view(shape)
            at += math.prod(shape)

    def neighbour_sum(self, t, paths, rows, h, pos, dst, src, sh):
        """[N, C, sum of 2 l3 + 1] over the edges given. rows: the paths' places among all of the layer's."""
        c, w, w3 = self.case, self.w, self.w["rad3_%d" % t].view(HIDDEN, -1, self.case["channels"])
        d = pos[src] - pos[dst] + sh
        r = d.norm(dim=-1)
        x, p = r / c["cutoff"], ENVELOPE
        fall = 1 - (p + 1) * (p + 2) / 2 * x ** p + p * (p + 2) * x ** (p + 1) - p * (p + 1) / 2 * x ** (p + 2)
        k = torch.arange(1, BASIS + 1, dtype=r.dtype, device=r.device) * math.pi
        basis = math.sqrt(2 / c["cutoff"]) * torch.sin(k * x[:, None]) / r[:, None] * fall[:, None]
        silu = torch.nn.functional.silu
        hidden = silu(silu(basis @ w["rad1_%d" % t]) @ w["rad2_%d" % t])
        y = _harmonics(d, c["lmax"])
        hj, out = h[src], []
        for row, (a, b, o) in zip(rows, paths):
            turn = torch.tensordot(y[:, b * b:(b + 1) ** 2], self.cg[a, b, o], ([1], [1]))  # [E, 2a+1, 2o+1]
            m = torch.bmm(hj[:, :, a * a:(a + 1) ** 2], turn) * (hidden @ w3[:, row])[:, :, None]
            out.append(torch.zeros(len(pos), *m.shape[1:], dtype=m.dtype, device=m.device).index_add(0, dst, m))
        return torch.cat(out, 2) / _neighbours(c["cutoff"])

    def atom_energies(self, pos, edges, charge=None):
        c, w = self.case, self.w
        dst, src, sh = edges
        silu, sl = torch.nn.functional.silu, lambda l: slice(l * l, (l + 1) ** 2)
        h = w["emb"][self.species][:, :, None]
        for t in range(1, c["layers"] + 1):
            every, product = _paths(c, t), c["correlation"] == 2
            orders = range(c["lmax"] + 1) if product else range(_top(c, t) + 1)
            keep = [i for i, p in enumerate(every) if p[2] in orders]
            paths = [every[i] for i in keep]
            step = int(4e8 / (c["channels"] * sum(2 * p[2] + 1 for p in paths)))
            if c["kind"] in ("train", "hessian", "hvp") or len(dst) <= step:
                sums = self.neighbour_sum(t, paths, keep, h, pos, dst, src, sh)
            else:
                sums = sum(torch.utils.checkpoint.checkpoint(self.neighbour_sum, t, paths, keep, h, pos, dst[i:i + step], src[i:i + step],
                                                             sh[i:i + step], use_reentrant=False) for i in range(0, len(dst), step))
            parts = sums.split([2 * p[2] + 1 for p in paths], 2)
            mixed = []
            for l in orders:
                rows = torch.cat([q for q, p in zip(parts, paths) if p[2] == l], 1)
                mixed.append(w["mix_%d_%d" % (t, l)].t() @ rows)
            if product:
                w1, w2, top = w["sym1_%d" % t][self.species], w["sym2_%d" % t][self.species], _top(c, t)
                b = [w1[:, l, :, None] * mixed[l] for l in range(top + 1)]
                for q, (l1, l2, o) in enumerate(_pairs(c, top)):
                    b[o] = b[o] + w2[:, q, :, None] * torch.einsum("abc,nka,nkb->nkc", self.cg[l1, l2, o], mixed[l1], mixed[l2])
                mixed = [w["lin_%d_%d" % (t, l)].t() @ b[l] for l in range(top + 1)]
            for l in range(len(mixed)):
                if l == 0 or t > 1:
                    mixed[l] = mixed[l] + w["self_%d_%d" % (t, l)].t() @ h[:, :, sl(l)]
            gate = torch.sigmoid(mixed[0])
            h = torch.cat([silu(mixed[0])] + [m * gate for m in mixed[1:]], 2)
        h = h[:, :, 0]
        e = (silu(h @ w["read1"]) @ w["read2"])[:, 0] + w["e0"][self.species]
        if charge is not None:
            q = h @ w["qhead"] + w["qbias"][self.species]
            size = torch.bincount(self.owner).to(q.dtype)
            q = q - ((torch.zeros_like(size).index_add(0, self.owner, q) - charge) / size)[self.owner]
            pair = []
            for a, b in zip(self.offsets[:-1], self.offsets[1:]):
                d = pos[None, a:b] - pos[a:b, None]
                other = ~torch.eye(b - a, dtype=torch.bool, device=self.dev)
                r = torch.where(other, d.square().sum(-1), 1.0).sqrt()
                x = r / SOFT_CORE
                core = torch.where(x < 1, 1 - 6 * x ** 5 + 15 * x ** 4 - 10 * x ** 3, 0.0)
                u = torch.where(other, core / (r * r + 1).sqrt() + (1 - core) / r, 0.0)
                pair.append(0.5 * K_E * q[a:b] * (u @ q[a:b]))
            e = e + torch.cat(pair)
        return e


def exact(case, seed):
    dev = torch.device("cuda")
    pos, species, cell, pbc, offsets, rng = _inputs(case, seed)
    flat = torch.tensor(_weights(case, seed), device=dev)
    x = torch.tensor(pos, device=dev, requires_grad=True)
    sums = lambda e: torch.zeros(len(offsets) - 1, dtype=e.dtype, device=dev).index_add(0, model.owner, e)  # noqa: E731

    if case["kind"] == "train":
        flat.requires_grad_(True)
    model = _Exact(case, flat, species, offsets)

    def forces(at):
        edges = _edge_list(at.detach(), cell, offsets, case["open"], case["cutoff"])
        at = at.detach().requires_grad_(True)
        e = model.atom_energies(at, edges, torch.tensor(_charges(case, rng), device=dev) if case["coulomb"] else None)
        (g,) = torch.autograd.grad(e.sum(), at)
        return sums(e.detach()), -g

    if case["kind"] in ("energy", "fresh"):
        e, f = forces(x)
        return {"energy": e, "forces": f}
    if case["kind"] == "md":
        v = torch.tensor(_velocities(species, rng), device=dev)
        kick = (0.5 * DT * ACCEL / torch.tensor(MASSES, dtype=v.dtype, device=dev))[model.species][:, None]
        at = x.detach()
        e, f = forces(at)
        for _ in range(case["steps"]):
            v = v + kick * f
            at = at + DT * v
            e, f = forces(at)
            v = v + kick * f
        return {"energy": e, "positions": at, "velocities": v, "forces": f}

    edges = _edge_list(x.detach(), cell, offsets, case["open"], case["cutoff"])
    e_atom = model.atom_energies(x, edges)
    (g,) = torch.autograd.grad(e_atom.sum(), x, create_graph=True)
    if case["kind"] == "train":
        e_ref, f_ref = _targets(case, species, offsets, rng)
        e_ref, f_ref = torch.tensor(e_ref, device=dev), torch.tensor(f_ref.astype(np.float32).astype(np.float64), device=dev)
        e = sums(e_atom)
        (grad,) = torch.autograd.grad((e - e_ref).square().mean() + (g + f_ref).square().mean(), flat)
        n = case["species"]
        return {"energy": e.detach(), "forces": -g.detach(), "grad": grad[:-n], "grad_e0": grad[-n:], "weights": flat.detach() - RATE * grad}
    if case["kind"] == "hvp":
        v = rng.standard_normal((case["vectors"], len(pos), 3)).astype(np.float32).astype(np.float64)
        return torch.stack([torch.autograd.grad(g, x, torch.tensor(k, device=dev), retain_graph=True)[0] for k in v])
    sizes, off = np.diff(offsets), offsets
    rows = []
    for k in range(3 * int(sizes.max())):
        v = torch.zeros_like(g)
        has = np.nonzero(sizes > k // 3)[0]
        v[off[has] + k // 3, k % 3] = 1.0
        rows.append(torch.autograd.grad(g, x, v, retain_graph=True)[0])
    rows = torch.stack(rows)
    return [rows[:3 * n, off[s]:off[s + 1]].reshape(3 * n, 3 * n).t() for s, n in enumerate(sizes)]
