"""One message-passing layer, forward and reverse, on synthetic destination-sorted edge lists of chosen sizes:
edge counts around the tile / block / launch boundaries of the edge kernels (needs a GPU)."""
import numpy as np
import pytest

import oracle
from hgnn_inputs.weights import init_layer_weights
from parity_util import TOL, relerr

pytestmark = pytest.mark.gpu


def _edges(rng, N, E):
    """E directed edges, sorted by destination, random sources and geometry; some atoms have no edge."""
    dst = np.sort(rng.integers(0, N, size=E)).astype(np.int32)
    col = rng.integers(0, N, size=E).astype(np.int32)
    rvec = (rng.standard_normal((E, 3)) * 1.5).astype(np.float32)
    d2 = (rvec.astype(np.float64) ** 2).sum(1).astype(np.float32)
    row_ptr = np.zeros(N + 1, np.int32)
    row_ptr[1:] = np.cumsum(np.bincount(dst, minlength=N))
    return row_ptr, dst, col, d2, rvec


def _run_layer(N, E, H, dtype, seed, lengths=None):
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(seed)
    row_ptr, dst, col, d2, rvec = _edges(rng, N, E)
    if lengths is not None:   # chosen row lengths instead of random destinations
        assert len(lengths) == N and sum(lengths) == E
        dst = np.repeat(np.arange(N, dtype=np.int32), lengths)
        row_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    colT_ptr, permT = oracle.transpose_plan(col, N)
    W = init_layer_weights(rng, H).astype(np.float32)
    h = rng.standard_normal((N, H)).astype(np.float32)
    v = (rng.standard_normal((N, 3)) * 0.3).astype(np.float32)
    gh = rng.standard_normal((N, H)).astype(np.float32)
    gv = rng.standard_normal((N, 3)).astype(np.float32)
    alpha = 1.0 / max(1.0, E / N)
    dt = {"f32": B.F32, "bf16": B.BF16}[dtype]
    dev = lambda a: torch.as_tensor(a).cuda()
    ws_b, saved_b = B.mp_layer_workspace_bytes(N, E, H, dt)
    ws = torch.empty(ws_b, dtype=torch.uint8, device="cuda")
    saved = torch.empty(saved_b, dtype=torch.uint8, device="cuda")
    t = dict(row_ptr=dev(row_ptr), dst=dev(dst), col=dev(col), d2=dev(d2), rvec=dev(rvec), colT=dev(colT_ptr),
             permT=dev(permT.astype(np.int32)), h=dev(h), v=dev(v), W=dev(W), gh=dev(gh), gv=dev(gv))
    h_out, v_out = torch.empty_like(t["h"]), torch.empty_like(t["v"])
    g_h, g_v, gW = torch.empty_like(t["h"]), torch.empty_like(t["v"]), torch.empty_like(t["W"])
    B.mp_layer_fwd(N, E, H, dt, alpha, t["row_ptr"], t["dst"], t["col"], t["d2"], t["rvec"], t["h"], t["v"], t["W"],
                   h_out, v_out, saved, ws)
    B.mp_layer_bwd(N, E, H, dt, alpha, t["row_ptr"], t["dst"], t["col"], t["d2"], t["rvec"], t["colT"], t["permT"],
                   t["h"], t["W"], saved, t["gh"], t["gv"], g_h, g_v, gW, ws)
    torch.cuda.synchronize()
    ho, vo, cache = oracle.mp_layer_fwd(h, v, dst, col, d2, rvec, W.astype(np.float64), alpha)
    gho, gvo, gWo = oracle.mp_layer_bwd(cache, gh, gv)
    tol = TOL[dtype]
    errs = dict(h=relerr(h_out.cpu().numpy(), ho), v=relerr(v_out.cpu().numpy(), vo),
                g_h=relerr(g_h.cpu().numpy(), gho), g_v=relerr(g_v.cpu().numpy(), gvo))
    got = oracle.unpack_layer(gW.cpu().numpy(), H)
    for k, want in gWo.items():
        errs["gW." + k] = relerr(got[k], want)
    print(f"layer N={N} E={E} H={H} {dtype}", {k: f"{e:.1e}" for k, e in errs.items()}, flush=True)
    for k, e in errs.items():
        assert e <= (tol["fwd"] if k in ("h", "v") else tol["grad"]), (k, e)


def _run_layer_unsaved(N, H, dtype, lengths):
    """Forward alone, without a saved buffer, against the oracle."""
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(N)
    E = sum(lengths)
    _, _, col, d2, rvec = _edges(rng, N, E)
    dst = np.repeat(np.arange(N, dtype=np.int32), lengths)
    row_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    W = init_layer_weights(rng, H).astype(np.float32)
    h = rng.standard_normal((N, H)).astype(np.float32)
    v = (rng.standard_normal((N, 3)) * 0.3).astype(np.float32)
    dt = {"f32": B.F32, "bf16": B.BF16}[dtype]
    ws = torch.empty(sum(B.mp_layer_workspace_bytes(N, E, H, dt)) + (1 << 20), dtype=torch.uint8, device="cuda")
    dev = lambda a: torch.as_tensor(a).cuda()
    h_out, v_out = torch.empty((N, H), device="cuda"), torch.empty((N, 3), device="cuda")
    B.mp_layer_fwd(N, E, H, dt, 0.25, dev(row_ptr), dev(dst), dev(col), dev(d2), dev(rvec), dev(h), dev(v), dev(W), h_out, v_out,
                   None, ws)
    torch.cuda.synchronize()
    ho, vo, _ = oracle.mp_layer_fwd(h, v, dst, col, d2, rvec, W.astype(np.float64), 0.25)
    assert relerr(h_out.cpu().numpy(), ho) <= TOL[dtype]["fwd"]
    assert relerr(v_out.cpu().numpy(), vo) <= TOL[dtype]["fwd"]


@pytest.mark.parametrize("H,dtype,N,E", [(256, "bf16", 700, 40001), (128, "f32", 300, 8191), (64, "bf16", 90, 1000),
                                         (256, "f32", 50, 0)])
def test_layer_without_saved_buffer_recomputes(H, dtype, N, E):
    """saved == NULL in both calls: the reverse pass recomputes what the forward pass would have kept; every output
    equals the saved-buffer calls bit for bit."""
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(H + E)
    row_ptr, dst, col, d2, rvec = _edges(rng, N, E)
    colT_ptr, permT = oracle.transpose_plan(col, N)
    dt = {"f32": B.F32, "bf16": B.BF16}[dtype]
    dev = lambda a: torch.as_tensor(a).cuda()
    t = dict(row_ptr=dev(row_ptr), dst=dev(dst), col=dev(col), d2=dev(d2), rvec=dev(rvec), colT=dev(colT_ptr),
             permT=dev(permT.astype(np.int32)), h=dev(rng.standard_normal((N, H)).astype(np.float32)),
             v=dev((rng.standard_normal((N, 3)) * 0.3).astype(np.float32)), W=dev(init_layer_weights(rng, H).astype(np.float32)),
             gh=dev(rng.standard_normal((N, H)).astype(np.float32)), gv=dev(rng.standard_normal((N, 3)).astype(np.float32)))
    alpha = 1.0 / max(1.0, E / N)
    ws_b, saved_b = B.mp_layer_workspace_bytes(N, E, H, dt)
    outs = []
    for keep in (True, False):
        ws = torch.empty(ws_b + (0 if keep else saved_b + 512 + 24 * N), dtype=torch.uint8, device="cuda")
        saved = torch.empty(saved_b, dtype=torch.uint8, device="cuda") if keep else None
        h_out, v_out = torch.full_like(t["h"], float("nan")), torch.full_like(t["v"], float("nan"))
        g_h, g_v, gW = torch.full_like(t["h"], float("nan")), torch.full_like(t["v"], float("nan")), torch.full_like(t["W"], float("nan"))
        B.mp_layer_fwd(N, E, H, dt, alpha, t["row_ptr"], t["dst"], t["col"], t["d2"], t["rvec"], t["h"], t["v"], t["W"],
                       h_out, v_out, saved, ws)
        ws.fill_(0x5a)             # nothing of the forward call survives in the workspace
        B.mp_layer_bwd(N, E, H, dt, alpha, t["row_ptr"], t["dst"], t["col"], t["d2"], t["rvec"], t["colT"], t["permT"],
                       t["h"], t["W"], saved, t["gh"], t["gv"], g_h, g_v, gW, ws)
        torch.cuda.synchronize()
        outs.append([x.cpu().numpy() for x in (h_out, v_out, g_h, g_v, gW)])
    for a, b in zip(*outs):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    # a workspace of the plain size is refused
    ws = torch.empty(ws_b, dtype=torch.uint8, device="cuda")
    with pytest.raises(B.HgnnError) as e:
        B.mp_layer_fwd(N, E, H, dt, alpha, t["row_ptr"], t["dst"], t["col"], t["d2"], t["rvec"], t["h"], t["v"], t["W"],
                       torch.empty_like(t["h"]), torch.empty_like(t["v"]), None, ws)
    assert e.value.code == -6


# With bf16 operands at H = 256 the W2 gradient has a branch-free launch over an even number of whole 32-edge blocks
# per workgroup (needs at least 2 x 256 blocks = 16384 edges) and a checking launch for the rest; the fused edge
# kernels work on 64-edge tiles with a masked last tile.
@pytest.mark.parametrize("E", [0, 1, 31, 32, 33, 63, 64, 65, 16383, 16384, 16385, 16384 + 32, 16384 + 63,
                               2 * 16384 + 97, 3 * 16384 - 1])
def test_layer_bf16_pairs_edge_counts(E):
    _run_layer(N=700, E=E, H=256, dtype="bf16", seed=E + 1)


# With bf16 pairs (H = 256) and with fp32 operands at H = 128 the reverse edge kernel sums g_z1 per destination out of
# its 64-edge tile, in 32-edge units: rows
# inside one unit are written directly, rows that cross units are added from per-unit partials by a second kernel,
# empty rows are zeroed there. Row lengths around the unit and tile sizes, at every alignment, with empty rows between.
@pytest.mark.parametrize("H,dtype", [(256, "bf16"), (128, "f32")])
@pytest.mark.parametrize("pattern", ["mixed", "aligned", "long", "ones", "one_row", "tail_rows_empty"])
def test_layer_row_lengths_with_destination_sums_in_the_edge_kernel(pattern, H, dtype, monkeypatch):
    rng = np.random.default_rng(7)
    if pattern == "mixed":
        lengths = [int(x) for x in rng.choice([0, 0, 1, 2, 5, 30, 31, 32, 33, 63, 64, 65, 96, 127, 129, 200], size=400)]
    elif pattern == "aligned":
        lengths = [32, 32, 64, 0, 32, 96, 0, 0, 64, 128, 32, 1, 31, 32] * 20
    elif pattern == "long":
        lengths = [700, 3, 0, 1025, 64, 5000, 1]
    elif pattern == "ones":
        lengths = [1] * 777
    elif pattern == "one_row":
        lengths = [0, 0, 4321, 0]
    else:
        lengths = [40, 17, 64, 7] + [0] * 50
    N, E = len(lengths), sum(lengths)
    _run_layer(N=N, E=E, H=H, dtype=dtype, seed=11, lengths=lengths)
    # the separate pass over g_z1 (kept for the calls that ask for the gradient with respect to d2) gives the same
    monkeypatch.setenv("HGNN_DSUM_IN_KERNEL", "0")
    _run_layer(N=N, E=E, H=H, dtype=dtype, seed=11, lengths=lengths)


# The same rows in the other layers whose edges are at most 128 words (H = 64: two of the four wavefronts walk the tile)
@pytest.mark.parametrize("H,dtype", [(64, "f32"), (64, "bf16"), (128, "bf16")])
@pytest.mark.parametrize("pattern", ["mixed", "aligned", "long", "ones", "one_row", "tail_rows_empty"])
def test_layer_row_lengths_with_destination_sums_of_narrow_layers(pattern, H, dtype, monkeypatch):
    test_layer_row_lengths_with_destination_sums_in_the_edge_kernel(pattern, H, dtype, monkeypatch)


@pytest.mark.parametrize("H,dtype,E", [(64, "f32", 1000), (64, "bf16", 4097), (128, "f32", 8191), (128, "bf16", 8193),
                                       (256, "f32", 4095)])
def test_layer_other_modes_edge_counts(H, dtype, E):
    _run_layer(N=300, E=E, H=H, dtype=dtype, seed=E)


# fp32 operands at H = 128: the W2 gradient recomputes a1 (two 16-edge chunks per 32-edge block,
# eight-chunk trips, grids rounded to multiples of eight workgroups, one ragged block at most)
@pytest.mark.parametrize("E", [0, 1, 15, 16, 17, 31, 32, 33, 255, 256, 257, 511, 16385, 3 * 16384 + 45])
def test_layer_f32_128_edge_counts(E):
    _run_layer(N=500, E=E, H=128, dtype="f32", seed=E + 7)


# The other layers whose W2 gradient the reverse edge kernel forms: at H = 64 two wavefronts share the rows of a tile and leave
# a partial each; no edge, a tile with an empty half, ragged tiles, more tiles than workgroups in flight
@pytest.mark.parametrize("H,dtype", [(64, "f32"), (64, "bf16"), (128, "bf16")])
@pytest.mark.parametrize("E", [0, 1, 31, 33, 63, 65, 8 * 64 - 1, 3 * 16384 + 45])
def test_layer_w2_gradient_in_the_edge_kernel(E, H, dtype):
    _run_layer(N=400, E=E, H=H, dtype=dtype, seed=E + 13)


# Atom counts around the split rules of the atom-level weight gradients (about 64 rows per split, at most one round
# of resident workgroups, whole workgroups per compute unit, a grid padded to groups of eight splits) and the row
# tiles of the atom-level products; few edges, so that the atom-level kernels decide the outcome.
@pytest.mark.parametrize("H,dtype,N", [(256, "bf16", 1), (256, "bf16", 255), (256, "bf16", 257), (256, "bf16", 2049),
                                       (256, "bf16", 16385), (256, "bf16", 33001), (128, "f32", 9000),
                                       (128, "bf16", 41000), (64, "f32", 70001), (256, "f32", 12345)])
def test_layer_atom_counts(H, dtype, N):
    _run_layer(N=N, E=3000, H=H, dtype=dtype, seed=N)


# Atom counts around the 16-row tiles of small batches and the largest batch that takes them (256 taller tiles)
@pytest.mark.parametrize("H,dtype,last", [(256, "bf16", 8192), (128, "f32", 8192), (128, "bf16", 8192), (64, "f32", 16384),
                                          (64, "bf16", 16384)])
@pytest.mark.parametrize("N", [2, 15, 16, 17, 33, 0, 1])
def test_layer_atom_counts_of_small_row_tiles(N, H, dtype, last):
    n = N if N > 1 else last + N
    _run_layer(N=n, E=3000 if N < 2 else 40 * n, H=H, dtype=dtype, seed=n)


# the last batch whose chains of products take 16-row tiles at H = 256, one per compute unit
@pytest.mark.parametrize("N", [4096, 4097])
def test_layer_atom_counts_of_short_chains(N):
    _run_layer(N=N, E=5000, H=256, dtype="bf16", seed=N)


# 2,000 rows around the mean lengths from which four wavefronts share a row (256 compute units): the sums of the forward pass, and
# those of the reverse pass
@pytest.mark.parametrize("H,dtype,E", [(64, "f32", 7812), (64, "bf16", 7813), (128, "f32", 7813), (256, "bf16", 3906),
                                       (256, "f32", 3907), (64, "bf16", 1953), (128, "bf16", 1954), (256, "bf16", 1954)])
def test_layer_rows_around_the_split_of_a_row(H, dtype, E):
    _run_layer(N=2000, E=E, H=H, dtype=dtype, seed=E + H)


# Batches whose first products run in one launch with the packing of the weights (up to 16 MB of weights read by all 16-row
# tiles, forward and reverse pass each with a line of its own) and the next larger ones
@pytest.mark.parametrize("H,dtype,N", [(64, "f32", 5456), (64, "bf16", 5457), (64, "f32", 8192), (64, "bf16", 8193),
                                       (128, "f32", 1360), (128, "bf16", 1361), (128, "f32", 2048), (128, "bf16", 2049)])
def test_layer_atom_counts_of_the_packing_launch(H, dtype, N):
    _run_layer(N=N, E=2000, H=H, dtype=dtype, seed=N)


# The reductions of a reverse pass share a launch with its last product (up to 80 MB of partials) or have one of their own: 256 partials
# of the W2 gradient are 64 MB at H = 256, five blocks per 64 atoms come on top
@pytest.mark.parametrize("H,dtype,N,E", [(256, "bf16", 300, 20000), (256, "bf16", 3000, 20000), (128, "f32", 17, 40000),
                                         (128, "bf16", 5000, 40000), (64, "f32", 16001, 40000), (256, "f32", 300, 20000)])
def test_layer_reductions_with_the_last_product(H, dtype, N, E):
    _run_layer(N=N, E=E, H=H, dtype=dtype, seed=N + H)


@pytest.mark.parametrize("H,dtype", [(64, "f32"), (128, "bf16")])
def test_layer_weights_at_any_alignment(H, dtype):
    """Weights at a 4-byte boundary: the reverse pass packs in a launch of its own, with the same bits as a result."""
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(H)
    N, E, dt = 100, 1500, {"f32": B.F32, "bf16": B.BF16}[dtype]
    row_ptr, dst, col, d2, rvec = _edges(rng, N, E)
    colT_ptr, permT = oracle.transpose_plan(col, N)
    W = torch.as_tensor(init_layer_weights(rng, H).astype(np.float32)).cuda()
    g = [torch.as_tensor(np.ascontiguousarray(a)).cuda() for a in (row_ptr, dst, col, d2, rvec)]
    plan = [torch.as_tensor(a.astype(np.int32)).cuda() for a in (colT_ptr, permT)]
    h, gh = (torch.as_tensor(rng.standard_normal((N, H)).astype(np.float32)).cuda() for _ in range(2))
    v, gv = (torch.as_tensor(rng.standard_normal((N, 3)).astype(np.float32)).cuda() for _ in range(2))
    outs = []
    for off in (0, 1, 2):
        w = torch.empty(W.numel() + 4, device="cuda")[off:off + W.numel()].copy_(W)
        assert w.data_ptr() % 16 == 4 * off
        ws_b, saved_b = B.mp_layer_workspace_bytes(N, E, H, dt)
        ws, saved = (torch.zeros(b, dtype=torch.uint8, device="cuda") for b in (ws_b, saved_b))
        out = [torch.empty_like(x) for x in (h, v, h, v, W)]
        B.mp_layer_fwd(N, E, H, dt, 0.1, *g, h, v, w, out[0], out[1], saved, ws)
        B.mp_layer_bwd(N, E, H, dt, 0.1, *g, *plan, h, w, saved, gh, gv, out[2], out[3], out[4], ws)
        outs.append([x.cpu().numpy().view(np.uint32) for x in out])
    for o in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(outs[0], o))


# Widths other than 64 / 128 / 256 take the fragment-GEMM path (bf16 operands, width padded to a multiple of 128, rows
# to 256): the paper's 866, widths on both sides of the padding steps, odd and small widths, edge counts around the
# 16 / 32 / 256-row groups.
@pytest.mark.parametrize("H,N,E", [(866, 300, 5000), (384, 200, 3001), (1024, 257, 777), (866, 40, 0), (320, 513, 9000),
                                   (500, 64, 256), (866, 5, 17), (333, 100, 1500), (257, 33, 700), (100, 80, 900), (24, 50, 300),
                                   # enough edges for the 256 x 128 tiles of the per-edge weight gradient: a ragged
                                   # last row tile (Hp = 384: 8 + 4 blocks), a single whole one (Hp = 256 is served
                                   # by the fused kernels, so 200 -> 256), and two whole ones (512)
                                   (320, 2000, 70001), (200, 1500, 66000), (512, 1800, 65536),
                                   # atoms whose edges span many 64-row strips of the forward per-atom sums (whole strips
                                   # in the middle), next to atoms without edges
                                   (384, 3, 1000), (866, 2, 300), (200, 40, 64), (200, 7, 65)])
def test_layer_wide_widths(H, N, E):
    _run_layer(N=N, E=E, H=H, dtype="bf16", seed=H + E)


# The weight gradient of W2 in 256 x 128 tiles whose last row tile sticks out (12 and 4 column blocks of 32 past the last whole
# tile), with ragged row blocks at the end of the edges
@pytest.mark.parametrize("H,N,E", [(300, 700, 65281), (641, 500, 65536 + 33)])
def test_layer_wide_weight_gradient_of_many_edges(H, N, E):
    _run_layer(N=N, E=E, H=H, dtype="bf16", seed=E)


# The forward edge kernel sums the messages of a strip of 64 rows (32 at H = 64) in its accumulators, eight rows at a time: atoms that end
# and begin at a strip's edge, inside its groups of eight, one after the other in one group, over two and many strips, a ragged last
# strip of one row, no edges at either end and in between. Without a saved buffer z2 is not stored.
@pytest.mark.parametrize("H,dtype", [(64, "f32"), (64, "bf16"), (128, "f32"), (128, "bf16"), (256, "f32")])
@pytest.mark.parametrize("lengths", [[0, 32, 32, 64, 1, 31, 0, 16, 8, 8, 40, 200, 0], [1, 1, 2, 3, 1, 5, 0, 19, 33, 63], [7, 57, 129]])
def test_layer_rows_at_strip_edges(H, dtype, lengths):
    _run_layer(N=len(lengths), E=sum(lengths), H=H, dtype=dtype, seed=H + len(lengths), lengths=lengths)
    _run_layer_unsaved(len(lengths), H, dtype, lengths)


# The last steps of those sums are taken by the chain of products up to one 32-row tile per compute unit (256), by a kernel of their own
# beyond: on both sides of the line, rows of every length up to three strips, a last 16-row tile of one row
@pytest.mark.parametrize("N", [8177, 8193])
def test_layer_rows_either_side_of_the_short_chains(N):
    lengths = np.random.default_rng(N).choice([0, 1, 3, 7, 70, 130], size=N, p=[.3, .3, .2, .18, .01, .01])
    _run_layer(N=N, E=int(lengths.sum()), H=128, dtype="bf16", seed=N, lengths=lengths.tolist())


# The per-atom sums of the fragment path's epilogues work on strips of 64 rows in tiles of 256: atoms that end and begin at a strip's
# and at a tile's edge, one atom of exactly a strip, atoms over two and over five strips, an atom of its own in a ragged last
# strip, atoms without edges at either end and in between
@pytest.mark.parametrize("H,lengths", [(300, [64, 64, 1, 63, 0, 64, 200, 56, 3]), (130, [0, 30, 300, 0, 0, 118, 5, 0]),
                                       (866, [256, 0, 256, 1]), (40, [10, 20, 34, 40, 24, 7, 121, 0]), (257, [255, 2, 255, 64, 63])])
def test_layer_wide_rows_at_strip_edges(H, lengths):
    _run_layer(N=len(lengths), E=sum(lengths), H=H, dtype="bf16", seed=H, lengths=lengths)


# ------------------------------------------------------------------------------------------------
# k edge attributes (radial basis of the edge length) in place of d2
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("E,k,rc", [(5000, 8, 5.0), (1, 2, 3.0), (777, 16, 6.0), (0, 4, 5.0)])
def test_edge_rbf_matches_the_oracle(E, k, rc):
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(E + k)
    d = rng.uniform(0.0, rc, size=E).astype(np.float32)
    if E > 3:
        d[:3] = (0.0, rc, np.float32(rc) * np.float32(0.999999))
    d2 = (d * d).astype(np.float32)
    attr = torch.full((max(E, 1), k), float("nan"), dtype=torch.float32, device="cuda")
    B.edge_rbf(E, torch.as_tensor(d2).cuda(), k, rc, attr)
    torch.cuda.synchronize()
    if E == 0:
        return
    want = oracle.edge_rbf(d2, k, rc)
    got = attr.cpu().numpy()[:E]
    assert np.all(np.isfinite(got))
    assert relerr(got, want) <= TOL["f32"]["fwd"]      # float32 arithmetic against the float64 definition


def _run_layer_attr(N, E, H, k, seed, rc=5.0, lengths=None):
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(seed)
    row_ptr, dst, col, d2, rvec = _edges(rng, N, E)
    if lengths is not None:   # chosen row lengths instead of random destinations
        assert len(lengths) == N and sum(lengths) == E
        dst = np.repeat(np.arange(N, dtype=np.int32), lengths)
        row_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    d2 = np.minimum(d2, np.float32(rc * rc))
    attr = oracle.edge_rbf(d2, k, rc).astype(np.float32) if k > 1 else d2[:, None].copy()
    colT_ptr, permT = oracle.transpose_plan(col, N)
    W = init_layer_weights(rng, H, k=k).astype(np.float32)
    h = rng.standard_normal((N, H)).astype(np.float32)
    v = (rng.standard_normal((N, 3)) * 0.3).astype(np.float32)
    gh = rng.standard_normal((N, H)).astype(np.float32)
    gv = rng.standard_normal((N, 3)).astype(np.float32)
    alpha = 1.0 / max(1.0, E / N)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    ws_b, saved_b = B.mp_layer_attr_workspace_bytes(N, E, H, k, B.BF16)
    ws = torch.empty(ws_b, dtype=torch.uint8, device="cuda")
    saved = torch.empty(saved_b, dtype=torch.uint8, device="cuda")
    t = dict(row_ptr=dev(row_ptr), dst=dev(dst), col=dev(col), attr=dev(attr), rvec=dev(rvec), colT=dev(colT_ptr),
             permT=dev(permT.astype(np.int32)), h=dev(h), v=dev(v), W=dev(W), gh=dev(gh), gv=dev(gv))
    h_out, v_out = torch.empty_like(t["h"]), torch.empty_like(t["v"])
    g_h, g_v = torch.empty_like(t["h"]), torch.empty_like(t["v"])
    gW = torch.full_like(t["W"], float("nan"))
    B.mp_layer_attr_fwd(N, E, H, k, B.BF16, alpha, t["row_ptr"], t["dst"], t["col"], t["attr"], t["rvec"], t["h"],
                        t["v"], t["W"], h_out, v_out, saved, ws)
    B.mp_layer_attr_bwd(N, E, H, k, B.BF16, alpha, t["row_ptr"], t["dst"], t["col"], t["attr"], t["rvec"], t["colT"],
                        t["permT"], t["h"], t["W"], saved, t["gh"], t["gv"], g_h, g_v, gW, ws)
    torch.cuda.synchronize()
    ho, vo, cache = oracle.mp_layer_fwd(h, v, dst, col, d2, rvec, W.astype(np.float64), alpha, attr=attr)
    gho, gvo, gWo = oracle.mp_layer_bwd(cache, gh, gv)
    tol = TOL["bf16"]
    errs = dict(h=relerr(h_out.cpu().numpy(), ho), v=relerr(v_out.cpu().numpy(), vo),
                g_h=relerr(g_h.cpu().numpy(), gho), g_v=relerr(g_v.cpu().numpy(), gvo))
    got_flat = gW.cpu().numpy()
    assert np.all(np.isfinite(got_flat)), "a gradient field was left unwritten"
    got = oracle.unpack_layer(got_flat, H, k)
    for name, want in gWo.items():
        errs["gW." + name] = relerr(got[name], want)
    errs["gW.W1[attr rows]"] = relerr(got["W1"][2 * H:], gWo["W1"][2 * H:])
    print(f"layer attr N={N} E={E} H={H} k={k}", {n: f"{e:.1e}" for n, e in errs.items()}, flush=True)
    for n, e in errs.items():
        assert e <= (tol["fwd"] if n in ("h", "v") else tol["grad"]), (n, e)


# H = 64 / 128 / 256 run on the fused kernels (attribute term on the matrix cores): tile boundaries (64 edges), the
# branch-free and the masked tile, every k residue of the four-slot staging, k = 16 (all slots) and k = 2
@pytest.mark.parametrize("N,E,H,k", [(300, 5000, 866, 8), (200, 3001, 256, 16), (100, 1500, 64, 4), (64, 700, 333, 3),
                                     (50, 0, 128, 5), (120, 2000, 300, 1), (700, 40001, 256, 8), (300, 64, 256, 2),
                                     (300, 8193, 128, 13), (90, 1000, 64, 16), (40, 63, 128, 7), (500, 20000, 256, 3)])
def test_layer_with_edge_attributes(N, E, H, k):
    _run_layer_attr(N=N, E=E, H=H, k=k, seed=H + E + k)


# ------------------------------------------------------------------------------------------------
# rows inside longer edge arrays, and values that are no numbers
# ------------------------------------------------------------------------------------------------
def _rows_problem(seed, H, k, lengths, lead=0, tail=0, pad_dst=0, two_sets=False):
    """Atoms of the given row lengths; `lead` and `tail` edges in front of row_ptr[0] and behind row_ptr[N], which belong to no row.
    two_sets: edges join atoms of even or of odd number only. Device arrays (dict) and the oracle's arguments for the edges of the rows."""
    import torch
    rng = np.random.default_rng(seed)
    N, E = len(lengths), sum(lengths)
    row_ptr, dst, col, d2, rvec = _edges(rng, N, lead + E + tail)
    dst = np.concatenate([np.full(lead, pad_dst), np.repeat(np.arange(N), lengths), np.full(tail, pad_dst)]).astype(np.int32)
    row_ptr = (lead + np.concatenate([[0], np.cumsum(lengths)])).astype(np.int32)
    if two_sets:
        assert N % 2 == 0
        col = col // 2 * 2 + dst % 2
    d2 = np.minimum(d2, np.float32(25.0))
    attr = oracle.edge_rbf(d2, k, 5.0).astype(np.float32) if k > 1 else d2[:, None].copy()
    colT_ptr, permT = oracle.transpose_plan(col[lead:lead + E], N)
    a = dict(row_ptr=row_ptr, dst=dst, col=col, attr=attr, rvec=rvec, colT=colT_ptr.astype(np.int32), permT=(permT + lead).astype(np.int32),
             h=rng.standard_normal((N, H)).astype(np.float32), v=(rng.standard_normal((N, 3)) * 0.3).astype(np.float32),
             W=init_layer_weights(rng, H, k=k).astype(np.float32), gh=rng.standard_normal((N, H)).astype(np.float32),
             gv=rng.standard_normal((N, 3)).astype(np.float32))
    return {n: torch.as_tensor(np.ascontiguousarray(x)).cuda() for n, x in a.items()}, a, slice(lead, lead + E)


def _rows_call(t, H, k, dtype, keep=True, backward=False, alpha=0.25):
    """h', v' (g_h, g_v) of the attribute entry points, or of the plain ones (k = 0); outputs and scratch start as NaN."""
    import torch
    from paper_2506_21788_amd import binding as B
    N, E, dt = t["h"].shape[0], t["dst"].numel(), {"f32": B.F32, "bf16": B.BF16}[dtype]
    bytes_ = B.mp_layer_attr_workspace_bytes(N, E, H, k, dt) if k else B.mp_layer_workspace_bytes(N, E, H, dt)
    ws, saved = (torch.full((n,), 0xff, dtype=torch.uint8, device="cuda") for n in (bytes_[0] + (0 if keep else bytes_[1] + 512 + 24 * N), bytes_[1]))
    attr = t["attr"] if k else t["attr"][:, 0].contiguous()
    out = [torch.full_like(t[n], float("nan")) for n in ("h", "v", "h", "v")]
    graph = (t["row_ptr"], t["dst"], t["col"], attr, t["rvec"])
    args = (N, E, H, k, dt, alpha) if k else (N, E, H, dt, alpha)
    (B.mp_layer_attr_fwd if k else B.mp_layer_fwd)(*args, *graph, t["h"], t["v"], t["W"], out[0], out[1], saved if keep else None, ws)
    if backward:
        (B.mp_layer_attr_bwd if k else B.mp_layer_bwd)(*args, *graph, t["colT"], t["permT"], t["h"], t["W"], saved, t["gh"], t["gv"],
                                                       out[2], out[3], torch.empty_like(t["W"]), ws)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in (out if backward else out[:2])]


# Edge arrays longer than the rows (so that one recorded graph serves several batches, or a slice of a batch): the forward pass
# leaves out the edges in front of row_ptr[0] and behind row_ptr[N], whatever atom they name. Last rows that end inside a group of
# eight, at a strip's and at a tile's edge; no edge of any row.
@pytest.mark.parametrize("H,dtype,k", [(64, "f32", 0), (64, "bf16", 0), (128, "f32", 0), (128, "bf16", 0), (256, "f32", 0), (256, "bf16", 0),
                                       (64, "bf16", 3), (128, "bf16", 16), (256, "bf16", 4), (300, "bf16", 0), (130, "bf16", 2)])
@pytest.mark.parametrize("lengths", [[5, 0, 40, 16], [30, 34, 0, 64, 128], [0, 0, 0]])
def test_layer_forward_leaves_out_edges_of_no_row(H, dtype, k, lengths):
    for lead, tail, pad_dst in [(0, 3, 0), (0, 200, 0), (0, 200, len(lengths) - 1), (9, 70, 1), (64, 0, 0)]:
        t, a, rows = _rows_problem(H + tail, H, max(k, 1), lengths, lead, tail, pad_dst)
        ho, vo, _ = oracle.mp_layer_fwd(a["h"], a["v"], a["dst"][rows], a["col"][rows], a["attr"][rows, 0], a["rvec"][rows],
                                        a["W"].astype(np.float64), 0.25, attr=a["attr"][rows])
        for keep in (True, False) if H in (64, 128, 256) else (True,):
            got = _rows_call(t, H, k, dtype, keep=keep)
            for x, want in zip(got, (ho, vo)):
                assert relerr(x, want) <= TOL[dtype]["fwd"], (lead, tail, pad_dst, keep)


# More tiles than workgroups in flight: one walks whole tiles and tiles with edges of no row in turn, the next tile's gathers under way
@pytest.mark.parametrize("H,dtype,k", [(64, "f32", 0), (128, "f32", 0), (128, "bf16", 0), (128, "bf16", 16), (256, "bf16", 4), (300, "bf16", 0)])
def test_layer_forward_of_many_edges_leaves_out_edges_of_no_row(H, dtype, k):
    lengths = np.random.default_rng(H).choice([0, 1, 17, 64, 200], size=2400).tolist()
    t, a, rows = _rows_problem(H, H, max(k, 1), lengths, 9, 30001, 5)
    ho, vo, _ = oracle.mp_layer_fwd(a["h"], a["v"], a["dst"][rows], a["col"][rows], a["attr"][rows, 0], a["rvec"][rows],
                                    a["W"].astype(np.float64), 0.02, attr=a["attr"][rows])
    got = _rows_call(t, H, k, dtype, alpha=0.02)
    assert relerr(got[0], ho) <= TOL[dtype]["fwd"] and relerr(got[1], vo) <= TOL[dtype]["fwd"]


# At other widths the reverse pass's sums per atom go by the rows as well (the weight gradients take every edge)
@pytest.mark.parametrize("H", [300, 130])
@pytest.mark.parametrize("lead,tail,pad_dst", [(0, 3, 0), (0, 200, 4), (9, 70, 1), (64, 0, 0)])
def test_layer_wide_reverse_sums_go_by_the_rows(H, lead, tail, pad_dst):
    t, a, rows = _rows_problem(H + tail, H, 1, [30, 34, 0, 64, 130], lead, tail, pad_dst)
    _, _, cache = oracle.mp_layer_fwd(a["h"], a["v"], a["dst"][rows], a["col"][rows], a["attr"][rows, 0], a["rvec"][rows],
                                      a["W"].astype(np.float64), 0.25)
    g_h, g_v, _ = oracle.mp_layer_bwd(cache, a["gh"], a["gv"])
    got = _rows_call(t, H, 0, "bf16", backward=True)
    assert relerr(got[2], g_h) <= TOL["bf16"]["grad"] and relerr(got[3], g_v) <= TOL["bf16"]["grad"]


# The sums of the forward edge kernel with edge attributes, an instance of its own, at the edges of its strips; at H = 256 their last
# steps are taken by the chain of products up to 4,096 atoms, by a kernel of their own beyond
@pytest.mark.parametrize("H,k", [(64, 4), (128, 5), (256, 16)])
@pytest.mark.parametrize("lengths", [[0, 32, 32, 64, 1, 31, 0, 16, 8, 8, 40, 200, 0], [1, 1, 2, 3, 1, 5, 0, 19, 33, 63], [7, 57, 129]])
def test_layer_attribute_rows_at_strip_edges(H, k, lengths):
    _run_layer_attr(N=len(lengths), E=sum(lengths), H=H, k=k, seed=H + len(lengths), lengths=lengths)


@pytest.mark.parametrize("N", [4081, 4097])
def test_layer_attribute_rows_either_side_of_the_short_chains(N):
    lengths = np.random.default_rng(N).choice([0, 1, 3, 7, 70, 130], size=N, p=[.3, .3, .2, .18, .01, .01])
    _run_layer_attr(N=N, E=int(lengths.sum()), H=256, k=4, seed=N, lengths=lengths.tolist())


# A value that is no number spoils the atoms that it reaches through edges and no other: every second atom has edges with every
# second atom only, so sums over runs next to one another in one strip, one group of eight rows and one wavefront stay apart
@pytest.mark.parametrize("H,dtype,k", [(64, "f32", 0), (64, "bf16", 0), (128, "f32", 0), (128, "bf16", 0), (256, "f32", 0), (256, "bf16", 0),
                                       (128, "bf16", 3), (256, "bf16", 4), (300, "bf16", 0), (300, "bf16", 3)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_layer_sums_of_other_atoms_stay_apart(H, dtype, k, value):
    lengths = [3, 2, 1, 5, 0, 4, 21, 28, 64, 1, 7, 80, 40, 2] * 3
    t, _, _ = _rows_problem(H, H, max(k, 1), lengths, two_sets=True)
    plain = _rows_call(t, H, k, dtype, backward=True)
    assert all(np.isfinite(x).all() for x in plain)
    for atom in (1, 6, 8, 25):
        other = np.arange(len(lengths)) % 2 != atom % 2
        bad = dict(t, h=t["h"].clone())
        bad["h"][atom, H // 2] = value
        for got, want in zip(_rows_call(bad, H, k, dtype, backward=True), plain):
            assert np.array_equal(got[other].view(np.uint32), want[other].view(np.uint32)), atom
        assert not np.isfinite(_rows_call(bad, H, k, dtype)[0][atom]).all()
