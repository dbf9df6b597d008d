"""Decoding heads of one hidden layer as wide as the features against the oracle (needs a GPU): both branches of every step of
the reverse pass share a launch, each with rows, groups and splits of its own."""
import numpy as np
import pytest

import oracle
from hgnn_inputs import deep_head_field_slices, deep_head_weight_count, init_deep_head_weights
from parity_util import TOL, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,dtype", [(64, "f32"), (128, "f32"), (128, "bf16"), (256, "bf16"), (256, "f32")])
@pytest.mark.parametrize("sizes,S,sources", [
    ([13], 1, (0,)),                          # one graph: one row tile each
    ([16, 17, 15, 1, 33], 3, (0, 2)),         # around the 16-row tiles, one source without graphs
    ([0, 0, 5, 0], 2, (0, 1)),                # graphs without atoms
    ([0, 0, 0], 2, (1,)),                     # no atom at all: the force branch has no rows
    ([1] * 300, 2, (0, 1)),                   # as many graphs as atoms
    ([512] * 16, 2, (0, 1)),                  # 8,192 atoms: the last batch of one launch for both products (H >= 128)
    ([512] * 16 + [1], 2, (0, 1)),
])
def test_plain_heads_match_the_oracle(sizes, S, sources, H, dtype):
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(H + len(sizes))
    graph_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    G, N, dt = len(sizes), int(graph_off[-1]), {"f32": B.F32, "bf16": B.BF16}[dtype]
    src = rng.choice(np.asarray(sources), size=G).astype(np.int32)
    h = rng.standard_normal((N, H)).astype(np.float32)
    v = (rng.standard_normal((N, 3)) * 0.5).astype(np.float32)
    p = oracle.pool_fwd(h, graph_off).astype(np.float32)
    Wh = init_deep_head_weights(rng, H, H, 1, S)
    gE, gF = rng.standard_normal(G).astype(np.float32), rng.standard_normal((N, 3)).astype(np.float32)
    t = {k: torch.as_tensor(a).cuda() for k, a in dict(off=graph_off, src=src, h=h, v=v, p=p, Wh=Wh, gE=gE, gF=gF).items()}
    plan = torch.empty(B.multihead_plan_ints(N, G, S), dtype=torch.int32, device="cuda")
    B.multihead_plan(N, G, S, t["off"], t["src"], plan)
    ws_b, sv_b = B.multihead_decode_workspace_bytes(N, G, H, H, S, dt)
    ws = torch.full((ws_b,), 0x5a, dtype=torch.uint8, device="cuda")
    sv = torch.empty(sv_b, dtype=torch.uint8, device="cuda")
    f32 = dict(dtype=torch.float32, device="cuda")
    energy, force = torch.empty(G, **f32), torch.empty((N, 3), **f32)
    g_p, g_h, g_v = torch.empty((G, H), **f32), torch.empty((N, H), **f32), torch.empty((N, 3), **f32)
    gWh = torch.full_like(t["Wh"], float("nan"))
    B.multihead_decode_fwd(N, G, H, H, S, dt, plan, t["p"], t["h"], t["v"], t["Wh"], energy, force, sv, ws)
    B.multihead_decode_bwd(N, G, H, H, S, dt, plan, t["p"], t["h"], t["v"], t["Wh"], sv, t["gE"], t["gF"], g_p, g_h, g_v,
                           gWh, ws)
    torch.cuda.synchronize()
    eo, fo, c = oracle.heads_deep_fwd(p, h, v, graph_off, src, Wh.astype(np.float64), H, 1, S)
    gpo, gho, gvo, gWo = oracle.heads_deep_bwd(c, gE, gF)
    errs = {k: relerr(a.cpu().numpy(), b) for k, a, b in [("energy", energy, eo), ("force", force, fo), ("g_p", g_p, gpo),
                                                          ("g_h", g_h, gho), ("g_v", g_v, gvo)] if b.size}
    got, per = gWh.cpu().numpy(), deep_head_weight_count(H, H, 1)
    assert np.all(np.isfinite(got)), "a gradient field was left unwritten"
    for s in range(S):
        for name, (lo, hi, _) in deep_head_field_slices(H, H, 1).items():
            want = gWo[s * per + lo:s * per + hi]
            if not want.any():
                assert not got[s * per + lo:s * per + hi].any(), (s, name)
            else:
                errs[f"s{s}.{name}"] = relerr(got[s * per + lo:s * per + hi], want)
    print(f"heads G={G} N={N} H={H} S={S} {dtype}", f"{max(errs.values()):.1e}", flush=True)
    for k, e in errs.items():
        assert e <= TOL[dtype]["fwd" if k in ("energy", "force") else "grad"], (k, e)


# groups count as tiles where the short row tiles are chosen, and a launch of its own is taken for either branch past the line
@pytest.mark.parametrize("H,dtype", [(64, "bf16"), (128, "f32"), (256, "bf16")])
@pytest.mark.parametrize("sizes,S", [([30] * 20, 237), ([30] * 20, 238), ([1] * 300, 247), ([3] * 200, 500), ([800, 1, 900] * 4, 33)])
def test_plain_heads_of_many_sources(sizes, S, H, dtype):
    test_plain_heads_match_the_oracle(sizes, S, tuple(range(0, S, 3)), H, dtype)


# the weight gradients of both branches in one launch (few sources, or few rows) or in one each
@pytest.mark.parametrize("H,dtype", [(64, "f32"), (128, "bf16"), (256, "bf16"), (256, "f32")])
@pytest.mark.parametrize("sizes,S", [([100] * 81, 4), ([100] * 81, 5), ([100] * 80, 5), ([4000, 1, 4000, 100], 6)])
def test_plain_heads_weight_gradients_of_both_branches(sizes, S, H, dtype):
    test_plain_heads_match_the_oracle(sizes, S, tuple(range(S)), H, dtype)


def test_more_sources_than_one_launch_reduces():
    """32,900 sources at H = 256: the weight gradients of the two branches no longer fit one launch of the reductions."""
    import torch
    from paper_2506_21788_amd import binding as B
    H, S, used = 256, 32900, [0, 17001, 32899]
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 61 GB of device memory")
    print("heads of", S, "sources", flush=True)
    rng = np.random.default_rng(8)
    per = deep_head_weight_count(H, H, 1)
    graph_off, src = np.array([0, 3, 4, 9], np.int32), np.array([2, 0, 1], np.int32)
    N, G = 9, 3
    h = rng.standard_normal((N, H)).astype(np.float32)
    v = rng.standard_normal((N, 3)).astype(np.float32)
    p = oracle.pool_fwd(h, graph_off).astype(np.float32)
    Wh = init_deep_head_weights(rng, H, H, 1, 3)
    gE, gF = rng.standard_normal(G).astype(np.float32), rng.standard_normal((N, 3)).astype(np.float32)
    f32 = dict(dtype=torch.float32, device="cuda")
    W, gW = torch.zeros((S, per), **f32), torch.full((S, per), float("nan"), **f32)
    W[used] = torch.as_tensor(Wh.reshape(3, per)).cuda()
    t = [torch.as_tensor(a).cuda() for a in (p, h, v)]
    plan = torch.empty(B.multihead_plan_ints(N, G, S), dtype=torch.int32, device="cuda")
    B.multihead_plan(N, G, S, torch.as_tensor(graph_off).cuda(), torch.tensor(used, dtype=torch.int32).cuda()[torch.as_tensor(src).long().cuda()], plan)
    ws_b, sv_b = B.multihead_decode_workspace_bytes(N, G, H, H, S, B.BF16)
    ws, sv = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (ws_b, sv_b))
    out = dict(energy=torch.empty(G, **f32), force=torch.empty((N, 3), **f32))
    grads = dict(g_p=torch.empty((G, H), **f32), g_h=torch.empty((N, H), **f32), g_v=torch.empty((N, 3), **f32))
    B.multihead_decode_fwd(N, G, H, H, S, B.BF16, plan, *t, W, *out.values(), sv, ws)
    B.multihead_decode_bwd(N, G, H, H, S, B.BF16, plan, *t, W, sv, torch.as_tensor(gE).cuda(), torch.as_tensor(gF).cuda(),
                           *grads.values(), gW, ws)
    eo, fo, c = oracle.heads_deep_fwd(p, h, v, graph_off, src, Wh.astype(np.float64), H, 1, 3)
    want = dict(zip(("energy", "force", "g_p", "g_h", "g_v", "gW"), (eo, fo, *oracle.heads_deep_bwd(c, gE, gF))))
    got = dict(out, **grads, gW=gW[used].ravel())
    for k, x in got.items():
        assert relerr(x.cpu().numpy(), want[k]) <= TOL["bf16"]["fwd"], k
    gW[used] = 0.0
    assert not any(bool((part != 0).any()) for part in gW.split(1000)), "a source without graphs has a gradient"


# the embedding at widths of one and several 256-column slabs: chunks of 2,048 atoms, lists of matches around the batches of eight
@pytest.mark.parametrize("N,H,elements", [(1, 300, 1), (9, 257, 1), (2049, 520, 1), (5000, 24, 40), (4096, 866, 3)])
def test_embedding_at_other_widths(N, H, elements):
    import torch
    from paper_2506_21788_amd import binding as B
    rng = np.random.default_rng(N + H)
    Z = rng.choice(rng.permutation(B.ZMAX)[:elements] + 1, size=N).astype(np.int32)
    emb = rng.standard_normal((B.ZMAX + 1, H)).astype(np.float32)
    g = rng.standard_normal((N, H)).astype(np.float32)
    tZ, te, tg = (torch.as_tensor(a).cuda() for a in (Z, emb, g))
    h, ge = torch.full_like(tg, float("nan")), torch.full_like(te, float("nan"))
    B.embed_fwd(N, H, tZ, te, h)
    ws = torch.empty(B.embed_bwd_workspace_bytes(N, H), dtype=torch.uint8, device="cuda")
    B.embed_bwd(N, H, tZ, tg, ge, ws)
    torch.cuda.synchronize()
    assert np.array_equal(h.cpu().numpy(), emb[Z])
    want = np.zeros((B.ZMAX + 1, H))
    np.add.at(want, Z, g.astype(np.float64))
    assert relerr(ge.cpu().numpy(), want) <= TOL["f32"]["grad"]


# whole rows as flat runs: one row up to 256 rows per workgroup, a last run that is short, more elements and rows than a launch
# holds threads; values are copied, or multiplied once (and added once): equal bits
@pytest.mark.parametrize("N,H", [(1, 1), (3, 1024), (1000, 65), (5000, 24), (300001, 24), (40001, 100), (9000, 333), (2049, 1023),
                                 (70_000_001, 1), (70_000_001, 3)])
def test_embedding_and_pooled_gradient_rows_at_other_widths(N, H):
    import torch
    from paper_2506_21788_amd import binding as B
    print("rows", N, H, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N + H)
    Z = torch.randint(0, B.ZMAX + 1, (N,), dtype=torch.int32, device="cuda", generator=gen)
    emb = torch.randn((B.ZMAX + 1, H), device="cuda", generator=gen)
    h = torch.full((N, H), float("nan"), device="cuda")
    B.embed_fwd(N, H, Z, emb, h)
    for a in range(0, N, 1 << 22):
        assert torch.equal(h[a:a + (1 << 22)], emb[Z[a:a + (1 << 22)].long()])
    off = torch.tensor([0, N // 3, N // 3, N - N // 7, N], dtype=torch.int32, device="cuda")   # one graph is empty
    G = 4
    g_p = torch.randn((G, H), device="cuda", generator=gen)
    graph = torch.repeat_interleave(torch.arange(G, device="cuda"), off.diff().long())
    for mode, scale in ((B.POOL_SUM, torch.ones(G, device="cuda")), (B.POOL_MEAN, 1.0 / off.diff().float())):
        want = g_p * scale[:, None]      # rounded before it is added
        got, before = torch.full((N, H), float("nan"), device="cuda"), h.clone()
        B.pool_by_graph_bwd(N, G, H, mode, off, g_p, got, False)
        B.pool_by_graph_bwd(N, G, H, mode, off, g_p, h, True)
        for a in range(0, N, 1 << 22):
            w = want[graph[a:a + (1 << 22)]]
            assert torch.equal(got[a:a + (1 << 22)], w)
            assert torch.equal(h[a:a + (1 << 22)], before[a:a + (1 << 22)] + w)


# the column slabs of the embedding's gradient: workgroups of their own for few chunks of atoms, dealt to fewer for many
@pytest.mark.parametrize("N,H", [(2048, 1000), (10241, 600), (22529, 1000), (45057, 300)])
def test_embedding_gradient_of_many_atoms_at_other_widths(N, H):
    test_embedding_at_other_widths(N, H, 20)


# the vector form: one chunk (whose sums are the result) and several, species of no, one and most atoms of a chunk, and a result
# at an address that takes no 16-byte stores
@pytest.mark.parametrize("N,H,elements", [(1, 64, 1), (2047, 128, 2), (2048, 256, 94), (2049, 64, 3), (6001, 256, 1), (9000, 128, 40)])
def test_embedding_gradient_at_vector_widths(N, H, elements):
    import torch
    from paper_2506_21788_amd import binding as B
    test_embedding_at_other_widths(N, H, elements)
    gen = torch.Generator(device="cuda").manual_seed(N)
    Z = torch.randint(1, elements + 1, (N,), dtype=torch.int32, device="cuda", generator=gen)
    g = torch.randn((N, H), device="cuda", generator=gen)
    ws = torch.empty(B.embed_bwd_workspace_bytes(N, H), dtype=torch.uint8, device="cuda")
    n, out = (B.ZMAX + 1) * H, []
    for off in (0, 1):
        buf = torch.full((n + 2,), float("nan"), device="cuda")
        B.embed_bwd(N, H, Z, g, buf[off:off + n], ws)
        assert bool(buf[:off].isnan().all()) and bool(buf[off + n:].isnan().all())
        out.append(buf[off:off + n])
    assert torch.equal(*out)
