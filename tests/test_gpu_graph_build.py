"""Radius graph and routing plan at the sizes where their kernels hand over to one another: batches of one workgroup per
graph against grid-wide binning, bins counted in LDS against memory, one-launch against block-sum scans, sources placed by
sixteen wavefronts against one."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from hgnn_inputs import concat_graphs, small_mixed_batch
from parity_util import assert_graph_equal
from test_gpu_parity import gpu_graph

pytestmark = pytest.mark.gpu


def repeated(b, times):
    """The batch's graphs over and over, and the oracle's graph of it put together from one copy."""
    graphs = [(b.pos[b.graph_off[g]:b.graph_off[g + 1]], b.Z[b.graph_off[g]:b.graph_off[g + 1]],
               b.cell[g] if b.pbc[g] else None) for g in range(b.G)]
    return concat_graphs(graphs * times)


def repeated_graph(one, b, times):
    r = np.arange(times, dtype=np.int64)
    ptr = lambda a, step: np.concatenate([(a[:-1].astype(np.int64)[None] + step * r[:, None]).ravel(),
                                          [a[-1] + step * (times - 1)]]).astype(np.int32)
    ids = lambda a, step: (a.astype(np.int64)[None] + step * r[:, None]).ravel().astype(np.int32)
    E, N = one["E"], b.N
    return dict(E=E * times, row_ptr=ptr(one["row_ptr"], E), colT_ptr=ptr(one["colT_ptr"], E),
                edge_graph_ptr=ptr(one["edge_graph_ptr"], E), dst=ids(one["dst"], N), col=ids(one["col"], N),
                permT=ids(one["permT"], E), shift=np.tile(one["shift"], (times, 1)), d2=np.tile(one["d2"], times),
                rvec=np.tile(one["rvec"], (times, 1)))


@pytest.mark.parametrize("atoms", [16384, 16385, 131072, 131073])
def test_graph_of_many_small_structures(atoms):
    print("many small structures", atoms, flush=True)
    b = small_mixed_batch(11, n_mol=6, n_cry=2)
    times = atoms // b.N
    rest = atoms - times * b.N
    one = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, 4.0)
    many = repeated(b, times)
    want = repeated_graph(one, b, times)
    if rest:     # fill up to the exact number with far-away single atoms: no edges
        lone = [(np.zeros((1, 3), np.float32), np.ones(1, np.int32))] * rest
        graphs = [(many.pos[many.graph_off[g]:many.graph_off[g + 1]], many.Z[many.graph_off[g]:many.graph_off[g + 1]],
                   many.cell[g] if many.pbc[g] else None) for g in range(many.G)]
        many = concat_graphs(graphs + lone)
        for k in ("row_ptr", "colT_ptr", "edge_graph_ptr"):
            want[k] = np.concatenate([want[k], np.full(rest, want["E"], np.int32)])
    assert many.N == atoms
    assert_graph_equal(gpu_graph(many, 4.0).to_numpy(), want)


@pytest.mark.parametrize("side", [40.0, 60.0])
def test_graph_of_a_sparse_structure_with_thousands_of_bins(side):
    """1,300 atoms in a large box: about 2,700 and 5,200 bins, on either side of what the workgroup counts in LDS."""
    print("sparse structure", side, flush=True)
    rng = np.random.default_rng(5)
    b = concat_graphs([(rng.uniform(0, side, (1300, 3)).astype(np.float32), np.ones(1300, np.int32))])
    rc = 2.85
    assert (np.floor(side / (1.001 * rc)) ** 3 > 4096) == (side > 50)
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, rc)
    assert want["E"] > 100
    assert_graph_equal(gpu_graph(b, rc).to_numpy(), want)


@pytest.mark.parametrize("G,S", [(1, 1), (63, 5), (65, 5), (1024, 64), (1025, 64), (2100, 64), (2100, 65)])
def test_routing_plan_sizes(G, S):
    import torch
    from paper_2506_21788_amd import binding as B
    print("routing plan", G, S, flush=True)
    rng = np.random.default_rng(G + S)
    sizes = rng.integers(0, 5, G)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    src = rng.integers(0, S, G).astype(np.int32)
    N = int(off[-1])
    plan = torch.full((B.multihead_plan_ints(N, G, S),), -7, dtype=torch.int32, device="cuda")
    B.multihead_plan(N, G, S, torch.as_tensor(off).cuda(), torch.as_tensor(src).cuda(), plan)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in B.plan_fields(plan, N, G, S).items()}
    # stable: graphs in batch order inside a source, atoms in graph order
    order = np.argsort(src, kind="stable")
    assert np.array_equal(got["graph_perm"], order)
    assert np.array_equal(got["grp_graph_ptr"], np.searchsorted(src[order], np.arange(S + 1)))
    atoms = np.concatenate([np.arange(off[g], off[g + 1]) for g in order]) if N else np.zeros(0)
    assert np.array_equal(got["atom_perm"], atoms)
    ag = np.repeat(np.arange(G), sizes)
    assert np.array_equal(got["atom_graph"], ag)
    assert np.array_equal(got["grp_atom_ptr"], np.searchsorted(src[ag][got["atom_perm"]], np.arange(S + 1)))


@pytest.mark.parametrize("off", [[0, 1, 0, 1], [0, 1, 0, 1, 0, 1, 0, 1], [0, 1, 1, 0, 1], [0, 1, 2], [-1, 1], [0, 0], [1, 1]])
def test_overlapping_sparse_graphs_are_refused(off):
    """Offsets (in units of the batch) that make graphs overlap, each of them with more bins than fit the LDS: refused,
    with nothing stored outside the workspace, and the workspace serves the next batch."""
    import torch
    from paper_2506_21788_amd import binding as B
    print("overlapping sparse graphs", off, flush=True)
    rng = np.random.default_rng(5)
    N, G, rc = 1300, len(off) - 1, 2.85
    b = concat_graphs([(rng.uniform(0, 60.0, (N, 3)).astype(np.float32), np.ones(N, np.int32))])
    pos = torch.as_tensor(b.pos).cuda()
    need, guard = B.radius_graph_workspace_bytes(N, G), 1 << 20
    ws = torch.full((need + guard,), 0x5A, dtype=torch.uint8, device="cuda")
    row_ptr = torch.full((N + 65,), -7, dtype=torch.int32, device="cuda")
    with pytest.raises(B.HgnnError) as e:
        B.radius_graph_count(N, G, pos, torch.tensor(off, dtype=torch.int32, device="cuda") * N, None, None, rc, ws, row_ptr)
    assert e.value.code == -3      # HGNN_ERR_BAD_OFFSETS
    assert bool((ws[need:] == 0x5A).all()) and bool((row_ptr[N + 1:] == -7).all())
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, rc)
    good = torch.tensor([0, N] + [N] * (G - 1), dtype=torch.int32, device="cuda")
    assert B.radius_graph_count(N, G, pos, good, None, None, rc, ws, row_ptr) == want["E"]
    assert np.array_equal(row_ptr[:N + 1].cpu().numpy(), want["row_ptr"])
    assert bool((ws[need:] == 0x5A).all())


def test_counting_and_routing_leave_a_drained_stream():
    """Both calls are documented to synchronise: at their return nothing is left to run, on whatever stream the results
    are read next. The routing of 40 million atoms takes a fraction of a millisecond after the source ids are checked."""
    import torch
    from paper_2506_21788_amd import binding as B
    other, mine = torch.cuda.Stream(), torch.cuda.Stream()
    N, G, S = 40_000_000, 2, 2
    print("routing plan", N, G, S, flush=True)
    off, src = torch.tensor([0, N // 2, N], dtype=torch.int32).cuda(), torch.tensor([1, 0], dtype=torch.int32).cuda()
    plan = torch.full((B.multihead_plan_ints(N, G, S),), -7, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(mine):
        B.multihead_plan(N, G, S, off, src, plan)
        assert mine.query()
    with torch.cuda.stream(other):
        f = B.plan_fields(plan, N, G, S)
        assert f["atom_perm"][[0, -1]].tolist() == [N // 2, N // 2 - 1] and f["atom_graph"][[0, -1]].tolist() == [0, 1]
        assert int(f["atom_perm"].min()) == 0
    del plan, f
    for N in (131072, 131073):          # degrees scanned by one launch, or by block sums
        print("counting", N, flush=True)
        pos = torch.zeros((N, 3), device="cuda")
        off = np.arange(0, N + 1, 2, dtype=np.int32)
        off[-1] = N                     # pairs of atoms on one place, and an odd atom joins the last
        sizes, G = np.diff(off), len(off) - 1
        want = torch.as_tensor(np.concatenate([[0], np.cumsum(np.repeat(sizes - 1, sizes))]).astype(np.int32)).cuda()
        off = torch.as_tensor(off).cuda()
        ws = torch.zeros(B.radius_graph_workspace_bytes(N, G), dtype=torch.uint8, device="cuda")
        row_ptr = torch.full((N + 1,), -7, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        for _ in range(20):
            with torch.cuda.stream(mine):
                row_ptr.fill_(-7)
                E = B.radius_graph_count(N, G, pos, off, None, None, 1.0, ws, row_ptr)
                assert mine.query()
            with torch.cuda.stream(other):
                assert torch.equal(row_ptr, want) and E == int(want[-1])


def test_refused_calls_keep_their_result_slot_until_nothing_can_post_to_it():
    """A call that ends with an error after its kernel was enqueued (here: an error that the caller left behind) returns
    with the stream drained, so that the kernel's result cannot land in the slot of the next call. Under capture the call is
    refused before anything is enqueued. Neither uses the slots up."""
    import ctypes
    import torch
    from paper_2506_21788_amd import binding as B
    hip = ctypes.CDLL(B.LIB_PATH)      # symbols of the runtime that the library calls
    b = small_mixed_batch(11, n_mol=6, n_cry=2)
    want = oracle.radius_graph(b.pos, b.graph_off, b.cell, b.pbc, 4.0)
    up = [torch.as_tensor(a).cuda() for a in (b.pos, b.graph_off, b.cell, b.pbc)]
    src = torch.as_tensor(b.source_id).cuda()
    S = int(b.source_id.max()) + 1
    plan = torch.zeros(B.multihead_plan_ints(b.N, b.G, S), dtype=torch.int32, device="cuda")
    ws = torch.zeros(B.radius_graph_workspace_bytes(b.N, b.G), dtype=torch.uint8, device="cuda")
    row_ptr = torch.zeros(b.N + 1, dtype=torch.int32, device="cuda")
    a = torch.rand((4096, 4096), device="cuda")
    slow, quick = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for k in range(3):
        print("left-over error", k, flush=True)
        with torch.cuda.stream(slow):
            for _ in range(10):
                c = a @ a
            assert not slow.query()
            assert hip.hipSetDevice(9999) != 0
            with pytest.raises(B.HgnnError, match="k_plan_graphs"):
                B.multihead_plan(b.N, b.G, S, up[1], src, plan)
            assert slow.query()
        with torch.cuda.stream(quick):
            assert B.radius_graph_count(b.N, b.G, *up, 4.0, ws, row_ptr) == want["E"]
            assert np.array_equal(row_ptr.cpu().numpy(), want["row_ptr"])
    del c
    print("capture", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.zero_()
        for _ in range(150):
            with pytest.raises(B.HgnnError, match="captured"):
                B.multihead_plan(b.N, b.G, S, up[1], src, plan)
            with pytest.raises(B.HgnnError, match="captured"):
                B.radius_graph_count(b.N, b.G, *up, 4.0, ws, row_ptr)
    graph.replay()
    assert B.radius_graph_count(b.N, b.G, *up, 4.0, ws, row_ptr) == want["E"]
    assert float(a.abs().max()) == 0.0


@pytest.mark.parametrize("sizes", [(4500,), (4501,), (4625, 4376), (9000, 1)])
def test_large_graphs_of_a_small_batch(sizes):
    """Few large graphs are binned by grid-wide kernels although the batch is small, on either side of the mean that decides.
    Each graph is one cluster of 125 atoms over and over (a lone atom at its end), at places that leave every difference of
    coordinates exact, so that its edges are the cluster's."""
    print("large graphs", sizes, flush=True)
    rng = np.random.default_rng(6)
    cluster = (rng.integers(0, 10 * 64, (125, 3)) / 64).astype(np.float32)
    one = oracle.radius_graph(cluster, np.array([0, 125], np.int32), np.zeros((1, 3, 3), np.float32), np.zeros(1, np.uint8), 4.0)
    place = np.stack(np.meshgrid(*[np.arange(5)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.float32) * 64
    graphs, parts, N, E = [], [], 0, 0
    for n in sizes:
        k = n // 125
        pos = np.concatenate([cluster + place[c] for c in range(k)] + [place[k:k + 1]] * (n % 125))
        graphs.append((pos, np.ones(n, np.int32)))
        w = repeated_graph(one, SimpleNamespace(N=125), k) if k else None
        parts.append((N, E, n, w))
        N, E = N + n, E + (w["E"] if k else 0)
    got = gpu_graph(concat_graphs(graphs), 4.0).to_numpy()
    assert got["E"] == E and E > 1000
    for n0, e0, n, w in parts:
        if w is None:
            continue
        e1, m = e0 + w["E"], n // 125 * 125
        for key, base in (("row_ptr", e0), ("colT_ptr", e0)):
            assert np.array_equal(got[key][n0:n0 + m + 1], w[key] + base), key
        for key, base in (("dst", n0), ("col", n0), ("permT", e0), ("shift", 0)):
            assert np.array_equal(got[key][e0:e1], w[key] + base), key
        assert np.array_equal(got["d2"][e0:e1].view(np.uint32), w["d2"].view(np.uint32))
        assert np.array_equal(got["rvec"][e0:e1].view(np.uint32), w["rvec"].view(np.uint32))


@pytest.mark.parametrize("atoms", [64, 6144, 6145, 12288, 12289])
def test_work_items_of_thin_cells_next_to_molecules(atoms):
    """Four, eight or sixteen destination atoms per work item by the size of the batch, only for graphs of many candidates:
    thin cells whose image blocks are streamed through the LDS (one with rows longer than the LDS row holds) between
    molecules that keep sixteen."""
    print("thin cells", atoms, flush=True)
    rng = np.random.default_rng(9)

    def cell(n, a):
        a = np.asarray(a)
        return (rng.random((n, 3)) @ a).astype(np.float32), rng.integers(1, 90, n).astype(np.int32), a.astype(np.float32)

    mol = lambda n: (rng.uniform(0, 6, (n, 3)).astype(np.float32), np.ones(n, np.int32))
    one_of = concat_graphs([cell(6, np.diag([2.5, 2.5, 2.5])), mol(21), cell(19, [[3, 0, 0], [1, 9, 0], [0, 2, 11]]), mol(1), mol(17)])
    rc = 6.0
    one = oracle.radius_graph(one_of.pos, one_of.graph_off, one_of.cell, one_of.pbc, rc)
    assert np.diff(one["row_ptr"]).max() > 256
    times, rest = divmod(atoms, one_of.N)
    many, want = repeated(one_of, times), repeated_graph(one, one_of, times)
    if rest:     # fill up to the exact number with single atoms: no edges
        graphs = [(many.pos[a:b], many.Z[a:b], many.cell[g] if many.pbc[g] else None)
                  for g, (a, b) in enumerate(zip(many.graph_off[:-1], many.graph_off[1:]))]
        many = concat_graphs(graphs + [(np.zeros((1, 3), np.float32), np.ones(1, np.int32))] * rest)
        for k in ("row_ptr", "colT_ptr", "edge_graph_ptr"):
            want[k] = np.concatenate([want[k], np.full(rest, want["E"], np.int32)])
    assert many.N == atoms
    assert_graph_equal(gpu_graph(many, rc).to_numpy(), want)


# The workgroup that bins a single graph also clears the counters, up to 16,384 of them (2,303 atoms): every byte of the workspace is
# dirty before each count, and what lies behind it stays as it is
@pytest.mark.parametrize("N", [1, 187, 2303, 2304])
def test_one_graph_clears_its_own_counters(N):
    import torch
    from paper_2506_21788_amd import binding as B
    print("one graph", N, flush=True)
    rng = np.random.default_rng(N)
    side = max(4.0, (N * 9.0) ** (1.0 / 3.0))
    a = np.array([[side, 0, 0], [0.3, side, 0], [0, -0.4, side]])
    one = concat_graphs([((rng.random((N, 3)) @ a).astype(np.float32), rng.integers(1, 90, N).astype(np.int32), a.astype(np.float32))])
    want = oracle.radius_graph(one.pos, one.graph_off, one.cell, one.pbc, 4.5)
    inputs = (N, 1, *(torch.as_tensor(x).cuda() for x in (one.pos, one.graph_off, one.cell, one.pbc)), 4.5)
    need, guard, E = B.radius_graph_workspace_bytes(N, 1), 1 << 16, want["E"]
    ws = torch.empty(need + guard, dtype=torch.uint8, device="cuda")
    tmp = torch.empty(8 * E + 16, dtype=torch.uint8, device="cuda")
    for dirt in (0x5A, 0xFF, 0x01):
        ws.fill_(dirt)
        out = {k: torch.full(want[k].shape, 77, dtype={"float32": torch.float32, "int8": torch.int8}.get(str(want[k].dtype), torch.int32),
                             device="cuda") for k in ("dst", "col", "shift", "d2", "rvec", "edge_graph_ptr", "colT_ptr", "permT")}
        row_ptr = torch.full((N + 1,), -7, dtype=torch.int32, device="cuda")
        assert B.radius_graph_count(*inputs, ws, row_ptr) == E
        B.radius_graph_fill(*inputs, ws, tmp, row_ptr, E, *out.values())
        assert_graph_equal(dict({k: v.cpu().numpy() for k, v in out.items()}, row_ptr=row_ptr.cpu().numpy(), E=E), want)
        assert bool((ws[need:] == dirt).all())


# atoms placed by the workgroup that places the graphs, or by a launch of their own
@pytest.mark.parametrize("N", [6144, 6145])
@pytest.mark.parametrize("G,S", [(1, 1), (1100, 64), (1100, 65), (7000, 5)])
def test_routing_plan_atom_counts(N, G, S):
    import torch
    from paper_2506_21788_amd import binding as B
    print("routing plan", N, G, S, flush=True)
    rng = np.random.default_rng(N + G + S)
    off = np.concatenate([[0], np.sort(rng.integers(0, N + 1, G - 1)), [N]]).astype(np.int32)   # some graphs are empty
    src = rng.integers(0, S, G).astype(np.int32)
    plan = torch.full((B.multihead_plan_ints(N, G, S),), -7, dtype=torch.int32, device="cuda")
    B.multihead_plan(N, G, S, torch.as_tensor(off).cuda(), torch.as_tensor(src).cuda(), plan)
    got = {k: v.cpu().numpy() for k, v in B.plan_fields(plan, N, G, S).items()}
    order = np.argsort(src, kind="stable")
    assert np.array_equal(got["graph_perm"], order)
    assert np.array_equal(got["atom_perm"], np.concatenate([np.arange(off[g], off[g + 1]) for g in order]))
    assert np.array_equal(got["atom_graph"], np.repeat(np.arange(G), np.diff(off)))
