"""Launch shapes of the matrix-core prefill that its plan treats apart: key ranges split with float32
partials (launches that can run whole), the same launches without a workspace, and waves
whose rows are all past the last (short suffixes), in every mode that has them.

Reference: float64 attention on the device over the same bf16 values; tolerance: the bf16 bar of the
parity tests (2e-2 absolute + 1e-2 relative, 1e-2 in the 2-norm)."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_28069_amd as pic  # noqa: E402

DEV = "cuda"


def _inputs(hq, hkv, d, ctx, n, seed=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    f = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16)
    B, cap = len(ctx), max(ctx) + n
    return dict(model=pic.Model.of(1, hq, hkv, d, "bf16", 5e5), q=f(B, n, hq, d), k=f(B, n, hkv, d), v=f(B, n, hkv, d),
                K=f(B, hkv, cap, d), V=f(B, hkv, cap, d), ctx=torch.tensor(ctx, dtype=torch.int32, device=DEV), B=B,
                cap=cap, n=n)


def _need(x, ctx):
    return pic.pic_prefill_workspace_bytes(x["model"], x["B"], x["n"], max(ctx))


def _prefill(x, ctx, ws):
    out = torch.full_like(x["q"], float("nan"))
    pic.pic_suffix_prefill_attn(x["model"], x["q"], x["k"], x["v"], x["K"], x["V"], x["B"], x["cap"], x["ctx"], max(ctx),
                                x["n"], out, ws)
    torch.cuda.synchronize()
    return out


def _check(x, ctx, out):
    hq, d = x["q"].shape[2:]
    errs = []
    for b, c in enumerate(ctx):
        n = x["n"]
        assert torch.equal(x["K"][b, :, c:c + n], x["k"][b].transpose(0, 1))
        assert torch.equal(x["V"][b, :, c:c + n], x["v"][b].transpose(0, 1))
        K, V = x["K"][b, :, :c + n].double(), x["V"][b, :, :c + n].double()
        rep = hq // K.shape[0]
        hidden = torch.arange(c + n, device=DEV)[None, :] > (c + torch.arange(n, device=DEV).repeat_interleave(rep))[:, None]
        for h in range(K.shape[0]):
            q = x["q"][b, :, h * rep:(h + 1) * rep].reshape(n * rep, d).double()
            s = (q @ K[h].t().contiguous() / math.sqrt(d)).masked_fill(hidden, -math.inf)
            ref = torch.softmax(s, -1) @ V[h]
            got = out[b, :, h * rep:(h + 1) * rep].reshape(n * rep, d).double()
            assert bool(((got - ref).abs() <= 2e-2 + 1e-2 * ref.abs()).all()), (b, h)
            errs.append(float((got - ref).norm() / ref.norm()))
            assert errs[-1] <= 1e-2, (b, h)
    return max(errs)


@pytest.mark.parametrize("hq,hkv,d,ctx,n", [
    (32, 8, 128, [4000, 3333, 100, 0, 4000, 4000, 4000, 64], 128),   # 128 units, uneven
    (32, 8, 64, [4096] * 16, 16),                                    # head_dim 64, one m-tile each
])
def test_split_with_float32_partials_and_whole_without_a_workspace(hq, hkv, d, ctx, n):
    x = _inputs(hq, hkv, d, ctx, n)
    need, rows = _need(x, ctx), x["B"] * n * hq
    assert need > 0 and need % (rows * (4 * d + 8)) == 0
    split = _check(x, ctx, _prefill(x, ctx, torch.full((need // 4,), float("nan"), device=DEV)))
    whole = _check(x, ctx, _prefill(x, ctx, None))
    short = _check(x, ctx, _prefill(x, ctx, torch.full((need // 8,), float("nan"), device=DEV)))
    assert split <= 1.05 * whole and short <= 1.05 * whole   # no precision lost to the split


# rows per (request, kv head) = tokens x (hq / hkv): one wave's 32, its edges, and the 256 of a workgroup
@pytest.mark.parametrize("hq,hkv,d,n", [(8, 2, 128, 1), (8, 2, 128, 8), (8, 2, 128, 9), (7, 1, 128, 36), (7, 1, 128, 37),
                                        (8, 2, 64, 33), (8, 1, 64, 5), (8, 2, 128, 65)])
@pytest.mark.parametrize("ctx", [[0, 1, 63, 64, 65, 200], [1500]])
def test_waves_without_rows(hq, hkv, d, n, ctx):
    x = _inputs(hq, hkv, d, ctx, n)
    _check(x, ctx, _prefill(x, ctx, torch.full((max(_need(x, ctx), 16) // 4,), float("nan"), device=DEV)))


@pytest.mark.parametrize("pairing", ["half", "interleaved"])
@pytest.mark.parametrize("d,n", [(128, 3), (128, 70), (64, 9)])
def test_waves_without_rows_in_every_mode(d, n, pairing):
    """Fused RoPE == turned first; zero-copy per key == composed; with a tile map within rounding."""
    hq, hkv = 8, 2
    lens = [100, 64, 150, 37, 128]
    T = sum(lens)
    offs = [sum(lens[:i]) for i in range(len(lens))]
    model = pic.Model.of(1, hq, hkv, d, "bf16", 5e5, pairing)
    blocks, ctx = pic.pic_plan_layout([[4, 2, 0, 1, 3, 2], [3]], offs, lens, [0] * 5, T)
    ctx = [int(c) for c in ctx]
    x = _inputs(hq, hkv, d, ctx, n, seed=3)
    mad = x["cap"]
    table = torch.empty(pic.pic_rope_table_bytes(model, mad) // 4, device=DEV)
    pic.pic_rope_table_init(model, mad, table)
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    pk, pv = (torch.randn((hkv, T, d), generator=g, device=DEV, dtype=torch.bfloat16) for _ in range(2))
    blk = torch.from_numpy(blocks.view("int32").copy()).to(DEV)
    pic.pic_compose(model, pk, pv, T, blk, len(blocks), table, mad, x["K"], x["V"], 2, x["cap"])
    ws = torch.empty(max(_need(x, ctx), 16), dtype=torch.uint8, device=DEV)
    # tokens turned by the call, against the same tokens turned first
    pos = (x["ctx"][:, None] + torch.arange(n, device=DEV, dtype=torch.int32)[None]).reshape(-1).contiguous()
    qt, kt = torch.empty_like(x["q"]), torch.empty_like(x["k"])
    pic.pic_rerotate_keys(model, x["q"], qt, 2 * n, hq, pos, table, mad)
    pic.pic_rerotate_keys(model, x["k"], kt, 2 * n, hkv, pos, table, mad)
    K2, V2 = x["K"].clone(), x["V"].clone()
    roped = torch.full_like(x["q"], float("nan"))
    pic.pic_suffix_prefill_attn_rope(model, x["q"], x["k"], x["v"], K2, V2, 2, x["cap"], x["ctx"], max(ctx), n, table, mad,
                                     roped, ws)
    x["q"], x["k"] = qt, kt
    want = _prefill(x, ctx, ws)
    _check(x, ctx, want)
    assert torch.equal(roped, want) and torch.equal(K2, x["K"]) and torch.equal(V2, x["V"])
    # straight from the pool
    src, dl = (torch.zeros((2, max(ctx)), dtype=torch.int32, device=DEV) for _ in range(2))
    tiles = torch.zeros((2, pic.pic_slot_map_tiles(max(ctx)), 2), dtype=torch.int32, device=DEV)
    pic.pic_build_slot_map(blk, len(blocks), 2, max(ctx), src, dl, tiles)
    for tm in (None, tiles):
        out = torch.full_like(qt, float("nan"))
        ck, cv = torch.zeros_like(x["K"]), torch.zeros_like(x["V"])
        pic.pic_paged_prefill_attn(model, pk, pv, T, src, dl, max(ctx), table, mad, qt, kt, x["v"], ck, cv, 2, x["cap"],
                                   x["ctx"], max(ctx), n, out, ws, tile_map=tm)
        torch.cuda.synchronize()
        if tm is None:
            assert torch.equal(out, want)
        else:
            assert float((out.double() - want.double()).norm() / want.double().norm()) <= 1e-2
