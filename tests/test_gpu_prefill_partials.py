"""Prefill launches split with float32 partials, whose rows leave the epilogue in two halves, in every
mode that has them: fused RoPE == turned first, zero-copy per key == composed (bit for bit, with the
same workspace), with a tile map within rounding; the composed call against float64 attention."""
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
