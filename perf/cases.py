"""The work whose speed is looked after: what a training or inference program has this library do, from one molecule to
a batch of large periodic cells.

A case is one call pattern on one batch of structures:

  train     radius graph, routing plan, forward and backward on a batch: the body of a training step
  predict   radius graph and forward only: energies and forces of structures on a trained model
  force     radius graph, forward and backward for the gradient of the energies with respect to the positions
            (conservative forces: molecular dynamics, relaxation)
  graph     the radius graph alone (data preparation)
  update    the AdamW update of every weight buffer

Structures are drawn here rather than with the rejection samplers of the tests, which take seconds for the large
batches: sites of a jittered grid, at the densities, sizes and element ranges of the benchmark's generators, with a
minimum distance and the same mean degree. Everything random comes from the seed.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2506_21788_amd import binding as B
from paper_2506_21788_amd.step import HotPath

BASE = {
    "mode": "train", "structures": "mixed", "graphs": 128, "atoms_lo": 5, "atoms_hi": 60,  # atoms per structure
    "cutoff": 5.0, "hidden": 256, "layers": 4, "sources": 5, "dtype": "bf16",
    "head_width": 0, "head_layers": 0,          # 0: one hidden layer as wide as the features
    "rbf": 0, "move": False,                    # radial-basis edge attributes (0: the squared length); moving atoms
}


def _case(**kw):
    return dict(BASE, **kw)


def listed():
    return [
        # one small molecule on the small model: an interactive or a dynamics call, all latency
        _case(name="predict_molecule", mode="predict", structures="molecules", graphs=1, atoms_lo=13, atoms_hi=13,
              hidden=64, layers=3, sources=1, dtype="f32"),
        # energies and forces of a validation batch of molecules
        _case(name="predict_molecules", mode="predict", structures="molecules", graphs=203, atoms_lo=10, atoms_hi=60,
              hidden=128, layers=4, dtype="bf16"),
        # one step of dynamics or relaxation of a crystal cell on conservative forces
        _case(name="force_crystal", mode="force", structures="crystals", graphs=1, atoms_lo=187, atoms_hi=187,
              cutoff=6.0, hidden=128, layers=4, sources=1, dtype="f32"),
        # the benchmark's configurations, a training step each: 32 small molecules, 128 molecules of five sources,
        # 64 crystals, the mixed five-source batch the benchmark is quoted on, and four large periodic cells
        _case(name="train_small_molecules", structures="molecules", graphs=32, atoms_lo=4, atoms_hi=20, hidden=64,
              layers=3, sources=1, dtype="f32"),
        _case(name="train_molecules", structures="molecules", graphs=128, atoms_lo=10, atoms_hi=60, hidden=128,
              layers=4, dtype="f32"),
        _case(name="train_crystals", structures="crystals", graphs=64, atoms_lo=8, atoms_hi=120, cutoff=6.0, layers=4,
              sources=1),
        _case(name="train_mixed", graphs=643, atoms_lo=5, atoms_hi=200, layers=6),
        _case(name="train_bulk", structures="bulk", graphs=4, atoms_lo=20000, atoms_hi=20000, cutoff=6.0, hidden=128,
              layers=3, sources=1, dtype="f32"),
        # the paper's model shape on its local batch of 128 structures (matrix-bound, odd widths)
        _case(name="train_wide", graphs=128, atoms_lo=5, atoms_hi=200, hidden=866, layers=4, head_width=889,
              head_layers=3),
        # atoms that move between layers, radial-basis edge attributes, position gradients: every option of a layer
        _case(name="train_moving", graphs=160, atoms_lo=5, atoms_hi=200, layers=4, rbf=16, move=True),
        # the radius graph of large cells alone
        _case(name="graph_bulk", mode="graph", structures="bulk", graphs=3, atoms_lo=21337, atoms_hi=21337, cutoff=6.0),
        # the weight update of the paper's model shape
        _case(name="update_wide", mode="update", hidden=866, layers=4, head_width=889, head_layers=3),
    ]


def draw(rng):
    """One more case: call pattern, kind and size of the batch, model width, depth, operand type and options."""
    mode = rng.choices(["train", "predict", "force", "graph", "update"], [10, 5, 3, 1, 1])[0]
    kind = rng.choices(["molecules", "crystals", "mixed", "bulk"], [4, 3, 4, 2])[0]
    width = rng.choices(["narrow", "wide"], [5, 1])[0]
    hidden = rng.choice([64, 128, 256]) if width == "narrow" else rng.randrange(300, 1001)
    dtype = rng.choice(["f32", "bf16"]) if hidden <= 128 else ("bf16" if hidden != 256 or rng.random() < 0.8 else "f32")
    c = _case(mode=mode, structures=kind, hidden=hidden, dtype=dtype, layers=rng.randrange(2, 7),
              sources=rng.randrange(1, 6), cutoff=rng.choice([4.5, 5.0, 5.5, 6.0]))
    if width == "wide" or (dtype == "bf16" and rng.random() < 0.2):
        c["head_layers"] = rng.randrange(1, 4)
        c["head_width"] = hidden if rng.random() < 0.5 else rng.randrange(64, 1001)
    if dtype == "bf16" and mode != "predict" and rng.random() < 0.25:
        c["rbf"] = rng.choice([4, 8, 16])
    if mode in ("train", "force") and rng.random() < 0.2:
        c["move"] = True
    # atoms of the batch, over the logarithm of its range
    total = math.exp(rng.uniform(math.log(12), math.log(60000)))
    if kind == "bulk":
        c["graphs"] = rng.randrange(1, 5)
        c["atoms_lo"] = c["atoms_hi"] = max(200, int(total / c["graphs"]))
    else:
        hi = min(rng.randrange(12, 61 if kind == "molecules" else 201), max(3, int(total)))
        c["atoms_lo"], c["atoms_hi"] = max(2, hi // rng.randrange(2, 11)), hi
        c["graphs"] = max(1, int(total / (_counts(dict(c, graphs=1000))[0] / 1000)))
    # a drawn case stays below the work of the largest listed one
    over = _load(c) / (0.7 * max(_load(dict(x)) for x in listed()))
    if over > 1.0:
        key = ["atoms_lo", "atoms_hi"] if kind == "bulk" else ["graphs"]
        c.update({x: max(1, int(c[x] / over)) for x in key})
    return c


def _load(case):
    """Elements of the edge tensors in bytes, and for the wide models the matrix work in the same unit: what the time of
    a training step goes with."""
    e = _counts(case)[1] * case["layers"] * case["hidden"] * (4 if case["dtype"] == "f32" else 2)
    option = 1.5 if case["rbf"] or case["move"] or (case["dtype"] == "f32" and case["hidden"] == 256) else 1.0
    return e * option * (max(1.0, case["hidden"] / 250) if case["hidden"] not in (64, 128, 256) else 1.0)


# ----------------------------------------------------------------------------------------------------------------------
# structures
def _sizes(case):
    """Atoms of every structure, spread evenly over the range (so that a batch of any seed has the same number), and
    whether it is a molecule (in a mixed batch three in five, of at most 60 atoms)."""
    G, lo, hi = case["graphs"], case["atoms_lo"], case["atoms_hi"]
    mol = {"molecules": G, "mixed": (3 * G + 2) // 5}.get(case["structures"], 0)
    mixed = case["structures"] == "mixed"

    def spread(n, lo, hi):
        return np.minimum(lo + ((np.arange(n) + 0.5) * (hi - lo + 1) / max(1, n)).astype(np.int64), hi)

    sizes = [spread(mol, min(lo, 30), min(hi, 60)) if mixed else spread(mol, lo, hi), spread(G - mol, lo, hi)]
    return np.concatenate(sizes), np.arange(G) < mol


def _sites(rng, n, m, gap):
    """n points of a jittered grid of m[0] x m[1] x m[2] sites, in fractions of the box; gap: the least distance of
    neighbouring points along an axis, in grid steps."""
    s = rng.permutation(m[0] * m[1] * m[2])[:n]
    p = np.stack([s // (m[1] * m[2]), s // m[2] % m[1], s % m[2]], axis=1) + gap / 2
    return (p + rng.random((n, 3)) * (1.0 - gap)) / np.asarray(m)


def _molecule(rng, n, share):
    """0.08 atoms per cubic Angstrom in a cubic box, at least 0.9 A apart; elements of organic molecules."""
    side = (n / 0.08) ** (1.0 / 3.0)
    m = max(1, math.ceil(n ** (1.0 / 3.0) - 1e-9))
    z = rng.choice(np.array([1, 6, 7, 8, 9, 16]), size=n)
    return side * _sites(rng, n, (m, m, m), min(1.0, 0.9 * m / side)), z, None


def _crystal(rng, n, share):
    """Triclinic cell: length ratios 4 : 15 at most, angles 60 to 120 degrees, 0.04 to 0.085 atoms per cubic Angstrom
    (share: where in that range, 0 to 1)."""
    while True:
        length = rng.uniform(4.0, 15.0, 3)
        ca, cb, cg = np.cos(np.deg2rad(rng.uniform(60.0, 120.0, 3)))
        g2 = 1.0 + 2.0 * ca * cb * cg - ca * ca - cb * cb - cg * cg
        if g2 > 0.25:
            break
    sg = math.sqrt(1.0 - cg * cg)
    cell = length[:, None] * np.array([[1.0, 0.0, 0.0], [cg, sg, 0.0], [cb, (ca - cb * cg) / sg, math.sqrt(g2) / sg]])
    cell *= (n / (0.04 + 0.045 * share) / np.linalg.det(cell)) ** (1.0 / 3.0)
    step = (np.linalg.det(cell) / n) ** (1.0 / 3.0)
    m = [max(1, math.ceil(v / step)) for v in np.linalg.norm(cell, axis=1)]
    while m[0] * m[1] * m[2] < n:
        m[int(np.argmax(np.linalg.norm(cell, axis=1) / m))] += 1
    return _sites(rng, n, m, 0.5) @ cell, rng.integers(1, 95, n), cell


def _bulk(rng, n, share):
    """Cubic periodic cell at 0.1 atoms per cubic Angstrom, at least 1 A apart."""
    side = (n / 0.1) ** (1.0 / 3.0)
    m = math.ceil(n ** (1.0 / 3.0) - 1e-9)
    return side * _sites(rng, n, (m, m, m), 1.0 * m / side), rng.integers(1, 31, n), side * np.eye(3)


def _batch(case, seed):
    rng = np.random.default_rng([seed, 1])
    sizes, molecule = _sizes(case)
    order = rng.permutation(len(sizes))
    sizes, molecule = sizes[order], molecule[order]
    G, N = len(sizes), int(sizes.sum())
    periodic = _bulk if case["structures"] == "bulk" else _crystal
    share = rng.permutation(np.arange(G) + 0.5) / G
    graphs = [(_molecule if mol else periodic)(rng, int(n), d) for n, mol, d in zip(sizes, molecule, share)]
    cell, pbc = np.zeros((G, 3, 3), np.float32), np.zeros(G, np.uint8)
    for g, (_, _, c) in enumerate(graphs):
        if c is not None:
            cell[g], pbc[g] = c, 1
    return SimpleNamespace(N=N, G=G, pos=np.concatenate([p for p, _, _ in graphs]).astype(np.float32),
                           Z=np.concatenate([z for _, z, _ in graphs]).astype(np.int32),
                           graph_off=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32), cell=cell, pbc=pbc,
                           source_id=rng.integers(0, case["sources"], G).astype(np.int32))


# ----------------------------------------------------------------------------------------------------------------------
# weights, in the layouts of the C header, as (shape, bound of the uniform values): 1/sqrt(inputs) for matrices and output
# vectors, 0.1 for biases
def _layer(case):
    H, k = case["hidden"], case["rbf"] or 1
    b, one, two = ((H,), 0.1), H ** -0.5, (2 * H) ** -0.5
    return [((2 * H + k, H), (2 * H + k) ** -0.5), b, ((H, H), one), b, ((H,), one), ((2 * H, H), two), b, ((H, H), one), b]


def _heads(case):
    H, Hh, D = case["hidden"], case["head_width"] or case["hidden"], case["head_layers"] or 1
    b, one = ((Hh,), 0.1), Hh ** -0.5
    head = [((H, Hh), H ** -0.5), b] + [((Hh, Hh), one), b] * (D - 1) + [((Hh,), one), ((1,), 0.1)]
    return head * (2 * case["sources"])


def _fill(rng, fields):
    return np.concatenate([(rng.random(math.prod(s), dtype=np.float32) * 2 - 1) * np.float32(b) for s, b in fields])


def prepare(case, seed):
    rng = np.random.default_rng([seed, 2])
    H = case["hidden"]
    if case["mode"] == "graph":
        b = _batch(case, seed)
        up = [torch.from_numpy(a).cuda() for a in (b.pos, b.graph_off, b.cell, b.pbc)]
        # edge arrays a loader keeps from batch to batch, with room for any batch of this kind
        room = 4096 + int((1.1 if b.N > 10000 else 3.0) * _counts(case)[1])
        i32, f32 = dict(dtype=torch.int32, device="cuda"), dict(dtype=torch.float32, device="cuda")
        edges = dict(dst=torch.zeros(room, **i32), col=torch.zeros(room, **i32),
                     shift=torch.zeros((room, 3), dtype=torch.int8, device="cuda"), d2=torch.zeros(room, **f32),
                     rvec=torch.zeros((room, 3), **f32), edge_graph_ptr=torch.zeros(b.G + 1, **i32),
                     colT_ptr=torch.zeros(b.N + 1, **i32), permT=torch.zeros(room, **i32))
        return SimpleNamespace(mode="graph", N=b.N, G=b.G, inputs=(*up, case["cutoff"]), edges=edges,
                               row_ptr=torch.zeros(b.N + 1, **i32),
                               ws=torch.zeros(B.radius_graph_workspace_bytes(b.N, b.G), dtype=torch.uint8, device="cuda"),
                               tmp=torch.zeros(8 * room, dtype=torch.uint8, device="cuda"))
    weights = [_fill(rng, _layer(case)) for _ in range(case["layers"])]
    heads = _fill(rng, _heads(case))
    emb = rng.standard_normal((B.ZMAX + 1, H), dtype=np.float32)
    if case["mode"] == "update":
        w = [torch.from_numpy(a.ravel()).cuda() for a in weights + [heads, emb]]
        gen = torch.Generator(device="cuda").manual_seed(seed)
        g = [1e-2 * torch.randn(a.numel(), device="cuda", generator=gen) for a in w]
        return SimpleNamespace(mode="update", w=w, g=g, m=[torch.zeros_like(a) for a in w],
                               v=[torch.zeros_like(a) for a in w], step=0)
    b = _batch(case, seed)
    hot = HotPath(b, case["cutoff"], H, case["layers"], case["sources"], case["dtype"], emb, weights, heads,
                  Hh=case["head_width"] or None, D=case["head_layers"] or None, rbf_k=case["rbf"] or None,
                  move=case["move"], pos_grad=case["mode"] == "force")
    # gradients of the loss with respect to the outputs; for conservative forces, of the total energy
    if case["mode"] == "force":
        gE, gF = -np.diff(b.graph_off).astype(np.float32), np.zeros((b.N, 3), np.float32)
    else:
        gE, gF = rng.standard_normal(b.G, dtype=np.float32), rng.standard_normal((b.N, 3), dtype=np.float32)
    return SimpleNamespace(mode=case["mode"], hot=hot, gE=torch.from_numpy(gE).cuda(), gF=torch.from_numpy(gF).cuda())


def run(state):
    if state.mode == "graph":
        s = state
        E = B.radius_graph_count(s.N, s.G, *s.inputs, s.ws, s.row_ptr)
        B.radius_graph_fill(s.N, s.G, *s.inputs, s.ws, s.tmp, s.row_ptr, E, **s.edges)
        return [E, s.row_ptr, s.edges]
    if state.mode == "update":
        state.step += 1
        for w, g, m, v in zip(state.w, state.g, state.m, state.v):
            B.adamw_step(w, g, m, v, state.step)
        return [state.w, state.m, state.v]
    hot = state.hot
    if state.mode == "predict":
        hot.build_plan()
        hot.build_graph()
        hot.forward()
        return [hot.energy, hot.force]
    if state.mode == "force":   # the structures stay the same, their atoms have moved
        hot.build_graph()
        hot.forward()
        hot.backward(state.gE, state.gF)
        return [hot.energy, hot.g_pos]
    hot.step(state.gE, state.gF)
    out = [hot.energy, hot.force, hot.gW, hot.gWhead, hot.g_emb]
    return out + [hot.g_pos] if hot.pos_grad else out


# ----------------------------------------------------------------------------------------------------------------------
def _counts(case):
    """Atoms and edges of a case (expected values over the seeds)."""
    n, molecule = _sizes(case)
    rc = case["cutoff"]
    ball = 4.0 / 3.0 * math.pi * rc ** 3
    # pairs of points of a cube that are closer than x of its side (x <= 1; nearly all beyond)
    x = np.minimum(rc / (n / 0.08) ** (1.0 / 3.0), 1.0)
    inside = n * (n - 1) * np.minimum(1.0, 4 / 3 * math.pi * x**3 - 1.5 * math.pi * x**4 + 1.6 * x**5 - x**6 / 6)
    periodic = n * ball * (0.1 if case["structures"] == "bulk" else 0.0625)
    return float(n.sum()), float(np.where(molecule, inside, periodic).sum())


def work(case):
    """Operations of the products (the first edge product once per atom and not per edge, the reverse pass twice the
    forward one, for positions alone once), and the bytes of inputs and outputs."""
    H, L, k = case["hidden"], case["layers"], case["rbf"] or 1
    Hh, D, S = case["head_width"] or H, case["head_layers"] or 1, case["sources"]
    layer = sum(math.prod(s) for s, _ in _layer(case))
    params = L * layer + sum(math.prod(s) for s, _ in _heads(case)) + (B.ZMAX + 1) * H
    if case["mode"] == "update":
        return {"bytes": 28.0 * params, "flops": 0.0}
    N, E = _counts(case)
    G = case["graphs"]
    inputs = 16.0 * N + 46.0 * G
    if case["mode"] == "graph":
        return {"bytes": inputs + 31.0 * E + 8.0 * N, "flops": 0.0}
    fwd = L * (10.0 * N * H * H + 2.0 * E * H * H + 2.0 * E * k * H) + 2.0 * (N + G) * (H * Hh + (D - 1) * Hh * Hh)
    if case["mode"] == "predict":
        return {"bytes": inputs + 4.0 * params + 4.0 * G + 12.0 * N, "flops": fwd}
    if case["mode"] == "force":
        return {"bytes": inputs + 4.0 * params + 8.0 * G + 12.0 * N, "flops": 2.0 * fwd}
    return {"bytes": inputs + 8.0 * params + 8.0 * G + 24.0 * N + 12.0 * N * case["move"], "flops": 3.0 * fwd}


def tolerance(case):
    """Measured against the float64 oracle on batches of up to 175,000 edges: with float32 operands at most 2.3e-6 in the
    norm (weight gradients: long sums with cancellation) and 1.3e-4 for one value, with bf16 operands 5.9e-3 and, for
    bias gradients near zero, up to a bias gradient's own size; four times that is stated."""
    if case["mode"] == "graph":
        return "exact"
    if case["mode"] == "update":
        return {"rel": 1e-6}
    return {"rel": 1e-5, "max": 6e-4} if case["dtype"] == "f32" else {"rel": 2e-2, "max": 0.9}
