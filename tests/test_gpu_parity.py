"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs."""
import sys

import numpy as np
import pytest

import oracle
from hgnn_inputs import concat_graphs, make_config, small_mixed_batch
from hgnn_inputs.structures import make_crystal, make_cubic_bulk

from parity_util import (TOL, assert_graph_equal, gpu_hotpath, oracle_graph, oracle_step,
                         problem_from_batch, problem_from_config, relerr, sub_batch)

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def gpu_graph(batch, rc):
    import torch
    from paper_2506_21788_amd.step import Graph, _dev
    g = Graph(_dev(batch.pos, torch.float32), _dev(batch.graph_off, torch.int32), _dev(batch.cell, torch.float32),
              _dev(batch.pbc, torch.uint8), rc)
    g.build()
    torch.cuda.synchronize()
    return g


# ------------------------------------------------------------------------------------------------
# radius graph: bit-exact
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("seed,rc", [(0, 5.0), (1, 4.0), (2, 6.0), (5, 3.0)])
def test_radius_graph_small_mixed(seed, rc):
    say("radius graph small mixed", seed, rc)
    b = small_mixed_batch(seed, n_mol=4, n_cry=4)
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, rc)
    got = gpu_graph(b, rc).to_numpy()
    assert_graph_equal(got, want)
    assert want["E"] > 100


@pytest.mark.parametrize("name", ["cfg1", "cfg2", "cfg3"])
def test_radius_graph_configs(name):
    say("radius graph", name)
    b, hp = make_config(name)
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, hp["rc"])
    got = gpu_graph(b, hp["rc"]).to_numpy()
    assert_graph_equal(got, want)


def test_radius_graph_edge_cases():
    say("radius graph edge cases")
    # single atoms, an isolated atom, an empty graph in the middle, a one-atom periodic cell
    pos1 = np.array([[0.0, 0, 0]], np.float32)
    mol = (np.array([[0, 0, 0], [1.0, 0, 0], [40.0, 0, 0]], np.float32), np.array([1, 6, 8], np.int32))
    cry = (pos1, np.array([3], np.int32), (np.eye(3) * 2.0).astype(np.float32))
    empty = (np.zeros((0, 3), np.float32), np.zeros(0, np.int32))
    b = concat_graphs([(pos1, np.array([1], np.int32)), mol, empty, cry, empty])
    for rc in (1.5, 2.0, 2.0001, 4.5):
        want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, rc)
        got = gpu_graph(b, rc).to_numpy()
        assert_graph_equal(got, want)
    # no atoms at all
    b0 = concat_graphs([empty])
    got = gpu_graph(b0, 3.0).to_numpy()
    assert got["E"] == 0 and got["row_ptr"].tolist() == [0]


def test_radius_graph_long_rows_and_many_images():
    """A dense small cell: rows of several hundred edges, up to 5 images per direction."""
    say("radius graph long rows")
    rng = np.random.default_rng(3)
    graphs = [make_crystal(rng, 12, 2.5, 3.5, 0.8, 1, 50, max_density=0.5) for _ in range(3)]
    b = concat_graphs(graphs)
    rc = 7.0
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, rc)
    assert np.diff(want["row_ptr"]).max() > 256
    got = gpu_graph(b, rc).to_numpy()
    assert_graph_equal(got, want)


def test_radius_graph_full_size_cfg5_sampled_rows():
    """Config 5 at its real size (4 x 20,000 atoms): every row pointer checked through sampled rows
    that the oracle computes one by one; global invariants checked everywhere."""
    say("radius graph cfg5 full size")
    b, hp = make_config("cfg5")
    g = gpu_graph(b, hp["rc"]).to_numpy()
    N = b.N
    deg = np.diff(g["row_ptr"])
    assert g["row_ptr"][0] == 0 and g["row_ptr"][-1] == g["E"]
    assert 85 < deg.mean() < 95
    rng = np.random.default_rng(0)
    rows = np.sort(rng.choice(N, size=64, replace=False))
    per = oracle.radius_graph_rows(b.pos, b.graph_off, b.cell, b.pbc, hp["rc"], rows)
    for i, (col, shift, d2, rvec) in zip(rows, per):
        e0, e1 = g["row_ptr"][i], g["row_ptr"][i + 1]
        assert np.array_equal(g["col"][e0:e1], col), i
        assert np.array_equal(g["shift"][e0:e1], shift), i
        assert np.array_equal(g["d2"][e0:e1].view(np.uint32), d2.view(np.uint32)), i
        assert np.array_equal(g["rvec"][e0:e1].view(np.uint32), rvec.view(np.uint32)), i
        assert np.all(g["dst"][e0:e1] == i)
    # invariants at any size
    assert np.array_equal(g["dst"], np.repeat(np.arange(N, dtype=np.int32), deg))
    key = g["dst"].astype(np.int64) * N + g["col"]
    assert np.all(np.diff(key) >= 0)
    ct, pt = oracle.transpose_plan(g["col"], N)
    assert np.array_equal(ct, g["colT_ptr"]) and np.array_equal(pt, g["permT"])
    assert np.array_equal(g["edge_graph_ptr"], g["row_ptr"][b.graph_off])


def test_radius_graph_error_paths():
    say("radius graph error paths")
    import torch
    from paper_2506_21788_amd import binding as B
    from paper_2506_21788_amd.step import _dev
    b = small_mixed_batch(0)
    N, G = b.N, b.G
    pos, cell, pbc = _dev(b.pos, torch.float32), _dev(b.cell, torch.float32), _dev(b.pbc, torch.uint8)
    ws = torch.empty(B.radius_graph_workspace_bytes(N, G), dtype=torch.uint8, device="cuda")
    row_ptr = torch.empty(N + 1, dtype=torch.int32, device="cuda")
    off = b.graph_off.copy()
    off[1], off[2] = off[2], off[1]
    if off[1] == off[2]:
        off[1] += 1
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, pos, _dev(off, torch.int32), cell, pbc, 4.0, ws, row_ptr)
    assert e.value.code == -3
    off = b.graph_off.copy()
    off[0] = 1
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, pos, _dev(off, torch.int32), cell, pbc, 4.0, ws, row_ptr)
    assert e.value.code == -3
    bad = b.cell.copy()
    gi = int(np.nonzero(b.pbc)[0][0])
    bad[gi][2] = bad[gi][1]
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, pos, _dev(b.graph_off, torch.int32), _dev(bad, torch.float32), pbc, 4.0, ws, row_ptr)
    assert e.value.code == -4
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, pos, _dev(b.graph_off, torch.int32), cell, pbc, -1.0, ws, row_ptr)
    assert e.value.code == -2
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, pos, _dev(b.graph_off, torch.int32), cell, pbc, 4.0, ws[:64], row_ptr)
    assert e.value.code == -6
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, None, _dev(b.graph_off, torch.int32), cell, pbc, 4.0, ws, row_ptr)
    assert e.value.code == -1
    # an atom of a periodic graph outside its cell (moved by one lattice vector): reported, not silently short of edges
    out = b.pos.copy()
    out[int(b.graph_off[gi])] += b.cell[gi][0]
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, _dev(out, torch.float32), _dev(b.graph_off, torch.int32), cell, pbc, 4.0, ws, row_ptr)
    assert e.value.code == -4 and "outside its cell" in str(e.value)
    # ... while a non-periodic graph may sit anywhere
    far = b.pos.copy()
    mol = int(np.nonzero(b.pbc == 0)[0][0])
    far[b.graph_off[mol]:b.graph_off[mol + 1]] += np.float32(1000.0)
    assert B.radius_graph_count(N, G, _dev(far, torch.float32), _dev(b.graph_off, torch.int32), cell, pbc, 4.0, ws, row_ptr) > 0
    # the good call still works afterwards
    assert B.radius_graph_count(N, G, pos, _dev(b.graph_off, torch.int32), cell, pbc, 4.0, ws, row_ptr) > 0


def test_radius_graph_fill_twice_after_one_count():
    """The filling call keeps no state of its own: a second fill after one count gives the same graph."""
    say("radius graph fill twice")
    import torch
    b = small_mixed_batch(4, n_mol=3, n_cry=3)
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, 4.5)
    g = gpu_graph(b, 4.5)
    assert_graph_equal(g.to_numpy(), want)
    from paper_2506_21788_amd import binding as B
    for t in (g.dst, g.col, g.permT, g.colT_ptr):
        t.fill_(-1)
    B.radius_graph_fill(g.N, g.G, g.pos, g.graph_off, g.cell, g.pbc, g.rc, g.ws, g.tmp, g.row_ptr, g.E, g.dst, g.col,
                        g.shift, g.d2, g.rvec, g.edge_graph_ptr, g.colT_ptr, g.permT)
    torch.cuda.synchronize()
    assert_graph_equal(g.to_numpy(), want)


def test_radius_graph_crowded_single_bin():
    """A dense cell thinner than two cutoffs: one bin whose 27 images hold several thousand candidates, which are
    streamed through the staging buffer in chunks."""
    say("radius graph crowded bin")
    rng = np.random.default_rng(8)
    graphs = [make_crystal(rng, 150, 7.0, 9.0, 0.7, 1, 50, max_density=0.4) for _ in range(2)]
    b = concat_graphs(graphs)
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, 5.0)
    got = gpu_graph(b, 5.0).to_numpy()
    assert_graph_equal(got, want)


# ------------------------------------------------------------------------------------------------
# whole step against the oracle
# ------------------------------------------------------------------------------------------------
def compare_step(P, tag, check_graph=True):
    import torch
    hp = P["hp"]
    tol = TOL[hp["dtype"]]
    og = oracle_graph(P)
    hpth = gpu_hotpath(P)
    hpth.build_graph()
    torch.cuda.synchronize()
    if check_graph:
        assert_graph_equal(hpth.graph.to_numpy(), og)
    alpha = hpth.alpha
    want = oracle_step(P, og, alpha, keep_layers=True)
    gE = torch.as_tensor(P["gE"]).cuda()
    gF = torch.as_tensor(P["gF"]).cuda()
    hpth.forward()
    hpth.backward(gE, gF)
    torch.cuda.synchronize()
    errs = {}
    for l in range(1, hp["L"] + 1):
        errs[f"h{l}"] = relerr(hpth.h[l].cpu().numpy(), want["hs"][l])
    errs["v"] = relerr(hpth.v[-1].cpu().numpy(), want["v"])
    errs["p"] = relerr(hpth.p.cpu().numpy(), want["p"])
    errs["energy"] = relerr(hpth.energy.cpu().numpy(), want["energy"])
    errs["force"] = relerr(hpth.force.cpu().numpy(), want["force"])
    gerrs = {"g_emb": relerr(hpth.g_emb.cpu().numpy(), want["g_emb"]),
             "g_heads": relerr(hpth.gWhead.cpu().numpy(), want["g_heads"]),
             "g_h0": relerr(hpth.g_h0.cpu().numpy(), want["g_h0"]),
             "g_v0": relerr(hpth.g_v0.cpu().numpy(), want["g_v0"])}
    from hgnn_inputs import layer_field_slices
    sl = layer_field_slices(hp["H"])
    for l in range(hp["L"]):
        got = hpth.gW[l].cpu().numpy()
        for name, (lo, hi, _) in sl.items():
            gerrs[f"gW{l}.{name}"] = relerr(got[lo:hi], want["g_layers"][l][lo:hi])
    say(tag, "N", P["batch"].N, "E", og["E"], "fwd", {k: f"{v:.2e}" for k, v in errs.items()})
    say(tag, "grad", {k: f"{v:.2e}" for k, v in gerrs.items()})
    for k, v in errs.items():
        assert v <= tol["fwd"], (tag, k, v)
    for k, v in gerrs.items():
        assert v <= tol["grad"], (tag, k, v)
    return hpth, want


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H", [64, 128, 256])
def test_step_small_mixed(H, dtype):
    say("step small mixed", H, dtype)
    b = small_mixed_batch(7, n_mol=5, n_cry=4, S=3, mol_atoms=(3, 40), cry_atoms=(2, 30))
    P = problem_from_batch(b, 4.5, H, 2, 3, dtype, seed=H)
    compare_step(P, f"small H={H} {dtype}")


def test_step_cfg1():
    say("step cfg1")
    compare_step(problem_from_config("cfg1"), "cfg1")


def test_step_cfg2():
    say("step cfg2")
    hpth, want = compare_step(problem_from_config("cfg2"), "cfg2")
    # routing plan is integer work: bit-exact
    from paper_2506_21788_amd import binding as B
    P = problem_from_config("cfg2")
    b = P["batch"]
    f = B.plan_fields(hpth.plan.cpu(), b.N, b.G, 5)
    ggp, gperm, gap, aperm = oracle.routing_plan(b.source_id, b.graph_off, 5)
    assert np.array_equal(f["grp_graph_ptr"].numpy(), ggp) and np.array_equal(f["graph_perm"].numpy(), gperm)
    assert np.array_equal(f["grp_atom_ptr"].numpy(), gap) and np.array_equal(f["atom_perm"].numpy(), aperm)


def test_step_cfg3_bf16():
    say("step cfg3")
    compare_step(problem_from_config("cfg3"), "cfg3")


def test_step_isolated_atoms_and_absent_source():
    """Rows with no edge (M = 0, v unchanged), a graph without any edge, a source with no graph."""
    say("step isolated/absent")
    import torch
    mol = (np.array([[0, 0, 0], [1.2, 0, 0], [40.0, 0, 0], [0, 1.1, 0.3]], np.float32), np.array([1, 6, 8, 7], np.int32))
    lone = (np.array([[0, 0, 0], [30.0, 0, 0]], np.float32), np.array([1, 1], np.int32))
    rng = np.random.default_rng(1)
    cry = make_crystal(rng, 6, 3.0, 5.0, 0.9, 1, 30, max_density=0.2)
    b = concat_graphs([mol, lone, cry], np.array([0, 3, 3], np.int32))
    P = problem_from_batch(b, 3.0, 64, 2, 4, "f32", seed=5)
    hpth, want = compare_step(P, "isolated")
    from hgnn_inputs import head_weight_count
    per = head_weight_count(64, 64)
    gh = hpth.gWhead.cpu().numpy()
    assert np.all(gh[per:3 * per] == 0.0) and np.any(gh[:per] != 0.0) and np.any(gh[3 * per:] != 0.0)


def test_step_is_bitwise_reproducible():
    say("step reproducible")
    import torch
    P = problem_from_config("cfg2")
    outs = []
    for _ in range(2):
        hpth = gpu_hotpath(P)
        hpth.build_graph()
        hpth.forward()
        hpth.backward(torch.as_tensor(P["gE"]).cuda(), torch.as_tensor(P["gF"]).cuda())
        torch.cuda.synchronize()
        outs.append([t.cpu().numpy().copy() for t in (hpth.energy, hpth.force, hpth.gWhead, hpth.g_emb, *hpth.gW)])
    for a, c in zip(*outs):
        assert np.array_equal(a.view(np.uint32), c.view(np.uint32))


def _paper_shape_small():
    b = small_mixed_batch(11, n_mol=5, n_cry=4, S=3, mol_atoms=(3, 40), cry_atoms=(2, 30))
    return problem_from_batch(b, 4.5, 866, 2, 3, "bf16", seed=866, Hh=889, D=3)


@pytest.mark.parametrize("which", ["cfg3", "paper-shape"])
def test_side_stream_on_and_off_give_the_same_bits(which):
    """Weight gradients may run on the library's side stream; keeping them on the caller's stream must not
    change a single bit (the sums have a fixed order either way). cfg3: bf16 pairs, i.e. the recomputing W2-gradient
    kernel with both of its launches (whole blocks, left-over and ragged blocks); paper-shape: the fragment path."""
    say("side stream on/off", which)
    import torch
    from paper_2506_21788_amd import binding as B
    P = problem_from_config("cfg3") if which == "cfg3" else _paper_shape_small()
    outs = []
    before = B.set_side_stream(True)
    try:
        for on in (True, False, None):
            B.set_side_stream(on)
            hpth = gpu_hotpath(P)
            hpth.build_graph()
            hpth.forward()
            hpth.backward(torch.as_tensor(P["gE"]).cuda(), torch.as_tensor(P["gF"]).cuda())
            torch.cuda.synchronize()
            outs.append([t.cpu().numpy().copy() for t in (hpth.energy, hpth.force, hpth.gWhead, hpth.g_emb, *hpth.gW)])
    finally:
        B.set_side_stream(before)
    for other in outs[1:]:
        for a, c in zip(outs[0], other):
            assert np.array_equal(a.view(np.uint32), c.view(np.uint32))


@pytest.mark.parametrize("name", ["cfg1", "cfg3", "paper-shape", "moving-atoms"])
def test_hip_graph_replays_match_eager_bitwise(name):
    """forward + backward recorded into a HIP graph: every replay, with eager work and synchronisations between
    the replays, gives the bits of the eager step."""
    say(f"hip graph {name}")
    import torch
    if name == "paper-shape":
        P = _paper_shape_small()
    elif name == "moving-atoms":   # per-layer geometry, radial basis, position gradients: their kernels and fills too
        b = small_mixed_batch(31, n_mol=5, n_cry=4, S=3, mol_atoms=(3, 40), cry_atoms=(2, 30))
        P = problem_from_batch(b, 4.5, 200, 3, 3, "bf16", seed=31, rbf_k=6, move=True)
    else:
        P = problem_from_config(name)
    gE, gF = torch.as_tensor(P["gE"]).cuda(), torch.as_tensor(P["gF"]).cuda()
    hpth = gpu_hotpath(P)
    hpth.build_graph()

    def outputs():
        torch.cuda.synchronize()
        extra = (hpth.g_pos,) if name == "moving-atoms" else ()
        return [t.cpu().numpy().copy() for t in (hpth.energy, hpth.force, hpth.gWhead, hpth.g_emb, hpth.g_h0, *hpth.gW, *extra)]

    hpth.forward()
    hpth.backward(gE, gF)
    want = outputs()
    graph = hpth.capture(gE, gF)
    for rep in range(3):
        for t in (hpth.energy, hpth.force, hpth.gWhead, hpth.g_emb, *hpth.gW):
            t.fill_(float("nan"))          # eager work between replays; also proves the replay rewrites everything
        torch.cuda.synchronize()
        graph.replay()
        got = outputs()
        for a, c in zip(want, got):
            assert np.array_equal(a.view(np.uint32), c.view(np.uint32)), rep
        hpth.forward()                       # an eager step in between
        hpth.backward(gE, gF)
        for a, c in zip(want, outputs()):
            assert np.array_equal(a.view(np.uint32), c.view(np.uint32)), rep


# ------------------------------------------------------------------------------------------------
# full sizes, in the launch configuration bench.py times
# ------------------------------------------------------------------------------------------------
# (configs 4, 5 and 6 at full size, every output and gradient field: tests/test_gpu_full_size.py)
def test_reduced_cfg5_backward():
    """Same density, cutoff, width and depth as config 5 on a cell the oracle can differentiate."""
    say("cfg5 reduced")
    rng = np.random.default_rng(0)
    graphs = [make_cubic_bulk(rng, 1500, 0.1, 1.0, 1, 30) for _ in range(2)]
    b = concat_graphs(graphs)
    P = problem_from_batch(b, 6.0, 128, 3, 1, "f32", seed=3)
    compare_step(P, "cfg5-reduced")


# ------------------------------------------------------------------------------------------------
# the paper's model shape: 866 hidden units, heads of three layers of 889 units (fragment-GEMM path)
# ------------------------------------------------------------------------------------------------
def test_step_small_mixed_paper_shape():
    say("step small mixed, H = 866, heads 3 x 889")
    compare_step(_paper_shape_small(), "small H=866 Hh=889 D=3 bf16")


def test_step_odd_width_plain_heads():
    """H = 100 with the plain heads of width 72: the layer takes the fragment path, the plain-heads entry points are
    served by the deep heads with one hidden layer."""
    say("step small mixed, H = 100, plain heads of width 72")
    from hgnn_inputs import init_head_weights
    b = small_mixed_batch(12, n_mol=4, n_cry=3, S=2, mol_atoms=(3, 30), cry_atoms=(2, 20))
    P = problem_from_batch(b, 4.5, 100, 2, 2, "bf16", seed=100)
    P["Wh"] = init_head_weights(np.random.default_rng(5), 100, 72, 2)
    P["hp"]["Hh"] = 72
    compare_step(P, "small H=100 Hh=72 bf16")


@pytest.mark.parametrize("H,k", [(128, 8), (866, 16)])
def test_step_with_radial_basis_edge_attributes(H, k):
    """Whole step with k radial-basis attributes per edge in place of d2 (every layer gradient field, the W1 rows
    that act on the attributes included)."""
    say("step small mixed with radial basis", H, k)
    b = small_mixed_batch(13, n_mol=5, n_cry=4, S=3, mol_atoms=(3, 40), cry_atoms=(2, 30))
    P = problem_from_batch(b, 4.5, H, 2, 3, "bf16", seed=H + k, rbf_k=k)
    import torch
    hp = P["hp"]
    tol = TOL["bf16"]
    og = oracle_graph(P)
    hpth = gpu_hotpath(P)
    hpth.build_graph()
    want = oracle_step(P, og, hpth.alpha, keep_layers=True)
    hpth.forward()
    hpth.backward(torch.as_tensor(P["gE"]).cuda(), torch.as_tensor(P["gF"]).cuda())
    torch.cuda.synchronize()
    errs = dict(h=relerr(hpth.h[-1].cpu().numpy(), want["h"]), energy=relerr(hpth.energy.cpu().numpy(), want["energy"]),
                force=relerr(hpth.force.cpu().numpy(), want["force"]))
    gerrs = dict(g_emb=relerr(hpth.g_emb.cpu().numpy(), want["g_emb"]),
                 g_heads=relerr(hpth.gWhead.cpu().numpy(), want["g_heads"]))
    from hgnn_inputs import layer_field_slices
    for l in range(hp["L"]):
        got = hpth.gW[l].cpu().numpy()
        for name, (lo, hi, _) in layer_field_slices(H, k).items():
            gerrs[f"gW{l}.{name}"] = relerr(got[lo:hi], want["g_layers"][l][lo:hi])
    say("rbf step", {n: f"{e:.2e}" for n, e in {**errs, **gerrs}.items()})
    for n, e in errs.items():
        assert e <= tol["fwd"], (n, e)
    for n, e in gerrs.items():
        assert e <= tol["grad"], (n, e)


# ------------------------------------------------------------------------------------------------
# pooling modes and many sources
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("H", [64, 256, 100])
def test_pool_sum_and_mean_overwrite_and_accumulate(H):
    """Both pooling modes, forward and reverse, with and without accumulation, on a batch with empty graphs."""
    say("pool modes", H)
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(H)
    sizes = [3, 0, 1, 70, 0, 257, 12]
    graph_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    N, G = int(graph_off[-1]), len(sizes)
    h = rng.standard_normal((N, H)).astype(np.float32)
    g_p = rng.standard_normal((G, H)).astype(np.float32)
    base = rng.standard_normal((N, H)).astype(np.float32)
    dev = lambda a: torch.as_tensor(a).cuda()
    for mode, mean in ((B.POOL_SUM, False), (B.POOL_MEAN, True)):
        p = torch.full((G, H), float("nan"), dtype=torch.float32, device="cuda")
        B.pool_by_graph_fwd(N, G, H, mode, dev(graph_off), dev(h), p)
        want = oracle.pool_fwd(h, graph_off, mean=mean)
        assert relerr(p.cpu().numpy(), want) <= TOL["f32"]["fwd"]
        assert np.all(p.cpu().numpy()[[1, 4]] == 0.0)
        want_g = oracle.pool_bwd(g_p, graph_off, N, mean=mean)
        g_h = torch.full((N, H), float("nan"), dtype=torch.float32, device="cuda")
        B.pool_by_graph_bwd(N, G, H, mode, dev(graph_off), dev(g_p), g_h, False)      # overwrite
        assert relerr(g_h.cpu().numpy(), want_g) <= TOL["f32"]["grad"]
        g_h = dev(base.copy())
        B.pool_by_graph_bwd(N, G, H, mode, dev(graph_off), dev(g_p), g_h, True)       # accumulate
        assert relerr(g_h.cpu().numpy(), base.astype(np.float64) + want_g) <= TOL["f32"]["grad"]


@pytest.mark.parametrize("H,sizes", [(128, [9000, 4097, 0, 5001]), (64, [12000, 1]), (256, [4096])])
def test_pool_few_large_graphs(H, sizes):
    """At 4096 atoms per graph and more the forward pooling splits a graph's columns over workgroups."""
    say("pool large graphs", H, sizes)
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(H + len(sizes))
    graph_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    N, G = int(graph_off[-1]), len(sizes)
    assert N >= 4096 * G
    h = rng.standard_normal((N, H)).astype(np.float32)
    for mode, mean in ((B.POOL_SUM, False), (B.POOL_MEAN, True)):
        p = torch.full((G, H), float("nan"), dtype=torch.float32, device="cuda")
        B.pool_by_graph_fwd(N, G, H, mode, torch.as_tensor(graph_off).cuda(), torch.as_tensor(h).cuda(), p)
        want = oracle.pool_fwd(h, graph_off, mean=mean)
        assert relerr(p.cpu().numpy(), want) <= TOL["f32"]["fwd"]
        for g, n in enumerate(sizes):
            if n == 0:
                assert np.all(p.cpu().numpy()[g] == 0.0)


@pytest.mark.parametrize("H,dtype,S", [(256, "bf16", 80), (128, "f32", 300), (64, "f32", 70)])
def test_step_many_sources(H, dtype, S):
    """More branches than the head weight gradient has compute units per split: most branches see no graph at all."""
    say("step many sources", H, dtype, S)
    b = small_mixed_batch(21, n_mol=6, n_cry=5, S=S, mol_atoms=(3, 30), cry_atoms=(2, 20))
    P = problem_from_batch(b, 4.5, H, 1, S, dtype, seed=S)
    compare_step(P, f"many sources H={H} {dtype} S={S}")


def test_kernel_classes_of_merged_launches():
    """The launches of small batches that do another class's work as well are classes of their own to the profile; where they are
    apart, the reductions of the heads count as column sums."""
    import torch
    from paper_2506_21788_amd import binding as B

    def launches(P):
        hot = gpu_hotpath(P)
        gE, gF = (torch.as_tensor(P[k]).cuda() for k in ("gE", "gF"))
        hot.step(gE, gF)
        side = B.set_side_stream(False)
        B.profile_begin((1 << B.profile_num_tags()) - 1)
        hot.step(gE, gF, with_graph=False)
        B.profile_end()
        B.set_side_stream(side)
        return {B.profile_tag_name(t): B.profile_read(t)[0] for t in range(B.profile_num_tags())}

    n = launches(problem_from_config("cfg1"))
    assert n["gemm_node_rows"] == 3 and n["gemm_node_reduce"] == 3 + 1 and n["seg_fwd"] == 0 and n["colsum"] == 1, n
    rng = np.random.default_rng(3)
    big = concat_graphs([(rng.uniform(0, 60.0, (9000, 3)).astype(np.float32), np.ones(9000, np.int32))])
    n = launches(problem_from_batch(big, 4.0, 128, 2, 1, "bf16"))
    assert n["gemm_node_rows"] == n["gemm_node_reduce"] == 0 and n["seg_fwd"] == 2 and n["colsum"] == 2, n
