"""Prefill launches split with float32 partials, whose rows leave the epilogue in two halves, in every
mode: fused RoPE == turned first, zero-copy per key == composed, inline tokens last == suffix (bit for
bit, with the same workspace), with a tile map within rounding; the composed call and inline layouts
against float64 attention."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_28069_amd as pic  # noqa: E402
from test_gpu_prefill_splits import DEV, _check, _inputs, _need, _prefill  # noqa: E402


# 128 and 136 units
@pytest.mark.parametrize("pairing", ["half", "interleaved"])
@pytest.mark.parametrize("hq,hkv,d,n,batch", [(32, 8, 128, 70, 8), (32, 8, 64, 9, 17)])
def test_modes_agree(hq, hkv, d, n, batch, pairing):
    lens = [100, 64, 150, 37, 128]
    requests = [[(b + 3 * i) % 5 for i in range(40 - b)] for b in range(batch)]
    T = sum(lens)
    offs = [sum(lens[:i]) for i in range(len(lens))]
    model = pic.Model.of(1, hq, hkv, d, "bf16", 5e5, pairing)
    blocks, ctx = pic.pic_plan_layout(requests, offs, lens, [0] * len(lens), T)
    ctx, B = [int(c) for c in ctx], len(requests)
    x = _inputs(hq, hkv, d, ctx, n, seed=3)
    mad = x["cap"]
    table = torch.empty(pic.pic_rope_table_bytes(model, mad) // 4, device=DEV)
    pic.pic_rope_table_init(model, mad, table)
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    pk, pv = (torch.randn((hkv, T, d), generator=g, device=DEV, dtype=torch.bfloat16) for _ in range(2))
    blk = torch.from_numpy(blocks.view("int32").copy()).to(DEV)
    pic.pic_compose(model, pk, pv, T, blk, len(blocks), table, mad, x["K"], x["V"], B, x["cap"])
    need = _need(x, ctx)
    assert need > 0 and need % (batch * n * hq * (4 * d + 8)) == 0
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device=DEV)
    # tokens turned by the call, against the same tokens turned first
    pos = (x["ctx"][:, None] + torch.arange(n, device=DEV, dtype=torch.int32)[None]).reshape(-1).contiguous()
    qt, kt = torch.empty_like(x["q"]), torch.empty_like(x["k"])
    pic.pic_rerotate_keys(model, x["q"], qt, B * n, hq, pos, table, mad)
    pic.pic_rerotate_keys(model, x["k"], kt, B * n, hkv, pos, table, mad)
    K2, V2 = x["K"].clone(), x["V"].clone()
    roped = torch.full_like(x["q"], float("nan"))
    pic.pic_suffix_prefill_attn_rope(model, x["q"], x["k"], x["v"], K2, V2, B, x["cap"], x["ctx"], max(ctx), n, table, mad,
                                     roped, ws)
    x["q"], x["k"] = qt, kt
    want = _prefill(x, ctx, ws)
    _check(x, ctx, want)
    assert torch.equal(roped, want) and torch.equal(K2, x["K"]) and torch.equal(V2, x["V"])
    # straight from the pool
    src, dl = (torch.zeros((B, max(ctx)), dtype=torch.int32, device=DEV) for _ in range(2))
    tiles = torch.zeros((B, pic.pic_slot_map_tiles(max(ctx)), 2), dtype=torch.int32, device=DEV)
    pic.pic_build_slot_map(blk, len(blocks), B, max(ctx), src, dl, tiles)
    for tm in (None, tiles):
        out = torch.full_like(qt, float("nan"))
        ck, cv = torch.zeros_like(x["K"]), torch.zeros_like(x["V"])
        pic.pic_paged_prefill_attn(model, pk, pv, T, src, dl, max(ctx), table, mad, qt, kt, x["v"], ck, cv, B, x["cap"],
                                   x["ctx"], max(ctx), n, out, ws, tile_map=tm)
        torch.cuda.synchronize()
        if tm is None:
            assert torch.equal(out, want)
        else:
            assert float((out.double() - want.double()).norm() / want.double().norm()) <= 1e-2


@pytest.mark.parametrize("hq,hkv,d,n,ctx", [(32, 8, 128, 70, [4000 - 100 * b for b in range(8)]), (28, 4, 128, 73, [4096] * 16),
                                            (32, 8, 64, 9, [3000 + 7 * b for b in range(16)])])
def test_inline_tokens_last_equal_the_suffix_call(hq, hkv, d, n, ctx):
    x = _inputs(hq, hkv, d, ctx, n)
    need, max_len = _need(x, ctx), max(ctx) + n
    assert need > 0 and need == pic.pic_frontier_workspace_bytes(x["model"], x["B"], n, max_len)
    pos = (x["ctx"][:, None] + torch.arange(n, dtype=torch.int32, device=DEV)[None]).contiguous()
    nv = torch.full((x["B"],), n, dtype=torch.int32, device=DEV)
    for ws in (torch.full((need // 4,), float("nan"), device=DEV), None):
        want = _prefill(x, ctx, ws)
        out = torch.full_like(want, float("nan"))
        K, V = x["K"].clone(), x["V"].clone()
        pic.pic_frontier_prefill_attn(x["model"], x["q"], x["k"], x["v"], K, V, x["B"], x["cap"], pos, nv, n, max_len, out, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(K, x["K"]) and torch.equal(V, x["V"])


@pytest.mark.parametrize("hq,hkv,d,n,batch", [(32, 8, 128, 128, 8), (28, 4, 128, 140, 8), (32, 8, 64, 40, 16)])
def test_inline_layouts(hq, hkv, d, n, batch):
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    f = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16)
    L = 4300
    pos = torch.stack([torch.randperm(L, generator=g, device=DEV)[:n].sort().values for _ in range(batch)]).int()
    nv = torch.tensor([n - 11 * (b % 3) for b in range(batch)], dtype=torch.int32, device=DEV)
    nv[1] = 0
    q, k, v, K, V = f(batch, n, hq, d), f(batch, n, hkv, d), f(batch, n, hkv, d), f(batch, hkv, L, d), f(batch, hkv, L, d)
    m = pic.Model.of(1, hq, hkv, d, "bf16", 5e5)
    need = pic.pic_frontier_workspace_bytes(m, batch, n, L)
    assert need > 0 and need % (batch * n * hq * (4 * d + 8)) == 0
    for ws in (torch.full((need // 4,), float("nan"), device=DEV), None):
        out = torch.full_like(q, 7.0)
        pic.pic_frontier_prefill_attn(m, q, k, v, K, V, batch, L, pos, nv, n, L, out, ws)
        torch.cuda.synchronize()
        rep = hq // hkv
        for b in range(batch):
            c = int(nv[b])
            assert bool((out[b, c:] == 7.0).all())
            if c == 0:
                continue
            p = pos[b, :c].long()
            hidden = torch.arange(L, device=DEV)[None] > p.repeat_interleave(rep)[:, None]
            for h in range(hkv):
                qq = q[b, :c, h * rep:(h + 1) * rep].reshape(c * rep, d).double()
                s = (qq @ K[b, h].double().t().contiguous() / d ** 0.5).masked_fill(hidden, -float("inf"))
                ref = torch.softmax(s, -1) @ V[b, h].double()
                got = out[b, :c, h * rep:(h + 1) * rep].reshape(c * rep, d).double()
                assert bool(((got - ref).abs() <= 2e-2 + 1e-2 * ref.abs()).all()), (b, h)
                assert float((got - ref).norm() / ref.norm()) <= 1e-2
