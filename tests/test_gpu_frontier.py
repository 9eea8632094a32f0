"""GPU parity of the general frontier layout (App. C.1; Sec. 2 canonical order P, D_1, S_1, ...,
D_m, S_m, Q with an inline prefix and inline spans between the documents): plan, compose and
frontier prefill through the C ABI against the oracle, then decode steps on the completed cache.

Tolerances as in test_gpu_parity: the plan and copied values bit-exact, bf16 keys within 1 bf16
ulp (+1e-5), attention within 2e-2 + 1e-2 |ref| with relative Frobenius error <= 1e-2 for bf16
and 1e-5 for float32.
"""
import numpy as np
import pytest
import torch

import paper_2607_28069_amd as pic
import synth
from oracle import pic_oracle as O
from synth import inputs as S

from gpu_path import (DEV, assert_attn_close, assert_keys_close, gpu_frontier, gpu_prefill, gpu_compose,
                      host, oracle_frontier, setup, setup_frontier, tdtype, to_dev)

pytestmark = pytest.mark.gpu


def _check_cache_and_out(r, out, n_inl):
    w = r.w
    ck, cv = host(r.dev["cache_k"][0]), host(r.dev["cache_v"][0])
    for b in range(w.batch):
        f = r.fmaps[b]
        ref, K, V = oracle_frontier(r, b)
        T = f.total_len
        assert np.array_equal(cv[b][:, :T].view(np.uint32), V.view(np.uint32)), b
        ip, cp = f.inline_pos, f.cached.logical_pos
        assert np.array_equal(ck[b][:, ip].view(np.uint32), K[:, ip].view(np.uint32)), b
        assert_keys_close(ck[b][:, cp], K[:, cp], w.dtype)
        n = int(n_inl[b])
        got = np.transpose(host(out[0, b, :n]), (1, 0, 2))
        assert_attn_close(got, np.transpose(ref, (1, 0, 2)), w.dtype)
        yield b, K, V


def _decode_after(r, steps, Ks, Vs):
    """Decode steps on the completed frontier cache vs the oracle, every request."""
    w, dt, d = r.w, tdtype(r.w), r.dev
    base = r.ctx.astype(np.int32)
    base_dev = torch.from_numpy(base).to(DEV)
    max_base = int(base.max())
    nbytes = pic.pic_decode_workspace_bytes(r.model, w.batch, max_base + steps, 0)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=DEV)
    dq = S.normal_f32(w, "dq_frontier", (steps, w.batch, w.n_q_heads, w.head_dim))
    dk = S.normal_f32(w, "dk_frontier", (steps, w.batch, w.n_kv_heads, w.head_dim))
    dv = S.normal_f32(w, "dv_frontier", (steps, w.batch, w.n_kv_heads, w.head_dim))
    if w.dtype == "bf16":
        dq, dk, dv = (S.bf16_bits_to_f32(S.f32_to_bf16_bits(x)) for x in (dq, dk, dv))
    lengths = [int(x) for x in base]
    for t in range(steps):
        out = torch.zeros((1, w.batch, w.n_q_heads, w.head_dim), dtype=dt, device=DEV)
        pic.pic_decode_attn(r.model, to_dev(dq[t][None], dt), to_dev(dk[t][None], dt), to_dev(dv[t][None], dt),
                            d["cache_k"], d["cache_v"], w.batch, r.cap, base_dev, t, max_base, out, ws)
        got = host(out[0])
        for b in range(w.batch):
            ref, Ks[b], Vs[b] = O.decode_step(Ks[b], Vs[b], lengths[b], dq[t][b], dk[t][b], dv[t][b])
            lengths[b] += 1
            assert_attn_close(got[b], ref, w.dtype)


@pytest.mark.parametrize("name", ["tiny_frontier_f32", "llama8b_frontier_1layer"])
def test_frontier_workloads(name):
    w = synth.get(name)
    r = setup_frontier(w)
    out, n_inl = gpu_frontier(r)
    torch.cuda.synchronize()
    assert list(n_inl) == [w.n_inline] * w.batch
    Ks, Vs = {}, {}
    for b, K, V in _check_cache_and_out(r, out, n_inl):
        Ks[b], Vs[b] = K, V
    print(f"[{name}] totals {[int(x) for x in r.ctx]}: cache and {w.n_inline} inline tokens ok", flush=True)
    _decode_after(r, 2, Ks, Vs)


def test_frontier_ragged_requests_and_split_keys():
    # Requests with different inline layouts (and so different inline counts, padded to the
    # largest): rows past a request's count stay untouched; the shape runs the key-range split
    # path (checked through the workspace the call asks for).
    w = synth.get("llama8b_frontier_1layer")
    # (at most 100 inline tokens: 2 m-tiles x 4 requests x 8 kv heads = 64 units, so the
    # launch is split over key ranges)
    items = [[-40, 0, -10, 1, -20, 2, -30], [3, 4, -64], [-5, 5, -3, 6, -1], [7, 8, 9, -100]]
    r = setup_frontier(w, items=items, n_inline_cap=100)
    m1 = r.model
    assert pic.pic_frontier_workspace_bytes(m1, w.batch, 100, int(r.ctx.max())) > 0
    out, n_inl = gpu_frontier(r, sentinel=7.0)
    torch.cuda.synchronize()
    assert list(n_inl) == [100, 64, 9, 100]
    for _ in _check_cache_and_out(r, out, n_inl):
        pass
    o = host(out[0])
    for b, n in enumerate(n_inl):
        assert np.all(o[b, n:] == 7.0), b
    print(f"[ragged] totals {[int(x) for x in r.ctx]} inline {[int(x) for x in n_inl]} ok", flush=True)


def test_frontier_call_equals_suffix_call_on_the_plain_layout():
    # The plain layout (documents back to back, query span last) through both entry points:
    # same cache, bit-identical attention outputs.
    w = synth.get("c2")
    r = setup(w)
    gpu_compose(r)
    out_a = gpu_prefill(r).clone()
    ck_a, cv_a = r.dev["cache_k"].clone(), r.dev["cache_v"].clone()
    lay = r.lay
    items = [list(req) + [-w.n_suffix] for req in lay.requests]
    blocks, total, inl, n_inl = pic.pic_plan_frontier(items, lay.doc_offset, lay.doc_len,
                                                      lay.doc_compile_pos, lay.pool_tokens)
    assert np.array_equal(total, r.ctx + w.n_suffix)
    assert np.array_equal(inl, r.ctx[:, None] + np.arange(w.n_suffix)[None, :])
    d = r.dev
    d["cache_k"].zero_()
    d["cache_v"].zero_()
    dt = tdtype(w)
    gpu_compose(r, blocks=blocks)
    out_b = torch.zeros_like(out_a)
    max_len = int(total.max())
    nbytes = pic.pic_frontier_workspace_bytes(r.model, w.batch, w.n_suffix, max_len)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=DEV)
    pic.pic_frontier_prefill_attn(r.model, d["q"], d["k_suf"], d["v_suf"], d["cache_k"], d["cache_v"],
                                  w.batch, r.cap, torch.from_numpy(inl).to(DEV),
                                  torch.from_numpy(n_inl).to(DEV), w.n_suffix, max_len, out_b, ws)
    torch.cuda.synchronize()
    assert torch.equal(d["cache_k"], ck_a) and torch.equal(d["cache_v"], cv_a)
    assert torch.equal(out_a, out_b)


# units per XCD (requests x kv heads / 8 x m-tiles): all pairs m-tile by m-tile (64), only the last
# round of pairs (144), pairs that do not divide over the XCDs (plain order), head_dim 64
@pytest.mark.parametrize("batch,hq,hkv,d,n", [(16, 32, 8, 128, 256), (16, 32, 8, 128, 570), (3, 28, 4, 128, 300),
                                              (8, 8, 2, 64, 200)])
def test_frontier_dispatch_orders_cover_every_row(batch, hq, hkv, d, n):
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    f = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16)
    max_len = 900
    pos = torch.stack([torch.randperm(max_len, generator=g, device=DEV)[:n].sort().values for _ in range(batch)]).int()
    nv = torch.tensor([n - 7 * (b % 3) for b in range(batch)], dtype=torch.int32, device=DEV)
    q, k, v, K, V = f(batch, n, hq, d), f(batch, n, hkv, d), f(batch, n, hkv, d), f(batch, hkv, max_len, d), f(batch, hkv, max_len, d)
    out = torch.full_like(q, 7.0)
    m = pic.Model.of(1, hq, hkv, d, "bf16", 5e5)
    ws = torch.empty(max(pic.pic_frontier_workspace_bytes(m, batch, n, max_len), 16), dtype=torch.uint8, device=DEV)
    pic.pic_frontier_prefill_attn(m, q, k, v, K, V, batch, max_len, pos, nv, n, max_len, out, ws)
    torch.cuda.synchronize()
    rep = hq // hkv
    for b in range(batch):
        c = int(nv[b])
        assert bool((out[b, c:] == 7.0).all())
        p = pos[b, :c].long()
        hidden = torch.arange(max_len, device=DEV)[None] > p.repeat_interleave(rep)[:, None]
        for h in range(hkv):
            assert torch.equal(K[b, h, p], k[b, :c, h]) and torch.equal(V[b, h, p], v[b, :c, h])
            qq = q[b, :c, h * rep:(h + 1) * rep].reshape(c * rep, d).double()
            s = (qq @ K[b, h].double().t().contiguous() / d ** 0.5).masked_fill(hidden, -float("inf"))
            ref = torch.softmax(s, -1) @ V[b, h].double()
            got = out[b, :c, h * rep:(h + 1) * rep].reshape(c * rep, d).double()
            assert bool(((got - ref).abs() <= 2e-2 + 1e-2 * ref.abs()).all()), (b, h)


# two and three m-tiles, past the line where only the last pairs go m-tile by m-tile (62 and 96 units
# per XCD), and four at the line (80) and past it (96)
@pytest.mark.parametrize("batch,hq,hkv,d,n", [(31, 64, 8, 128, 57), (32, 32, 8, 128, 190), (20, 32, 8, 64, 250), (24, 32, 8, 128, 250)])
def test_frontier_dispatch_orders_of_few_m_tiles(batch, hq, hkv, d, n):
    test_frontier_dispatch_orders_cover_every_row(batch, hq, hkv, d, n)


# up to 64 rows per (request, kv head) are stored from the registers, more go through LDS
@pytest.mark.parametrize("batch,hq,hkv,d,n", [(4, 8, 2, 128, 16), (4, 8, 2, 64, 16), (4, 8, 2, 128, 17), (5, 4, 2, 128, 32)])
def test_frontier_of_few_rows(batch, hq, hkv, d, n):
    test_frontier_dispatch_orders_cover_every_row(batch, hq, hkv, d, n)
