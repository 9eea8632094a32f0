"""float32 attention at the edges of its tiling: 16-key tiles, 16- and 32-row workgroups, eight
waves that take tiles in turn, the first tile a row sees only in part, rows past the last.

Tolerance: the float32 bar of the parity tests, 1e-5 absolute (N(0, 1) values, sums of at most a
few hundred terms, unit-scale outputs)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_28069_amd as pic          # noqa: E402
from oracle import pic_oracle as O          # noqa: E402

DEV = "cuda"


def _run(hq, hkv, d, ctx, n_q, seed=0, plant=None):
    """Suffix prefill over random caches (n_q None: one decode step): host arrays, out, caches."""
    rng = np.random.default_rng(seed)
    B, decode = len(ctx), n_q is None
    n = 1 if decode else n_q
    cap = max(ctx) + n + 1
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    h = dict(K=f(B, hkv, cap, d), V=f(B, hkv, cap, d), q=f(B, n, hq, d), k=f(B, n, hkv, d), v=f(B, n, hkv, d))
    if plant:
        plant(h)
    t = {a: torch.from_numpy(x.copy()).to(DEV) for a, x in h.items()}
    model = pic.Model.of(1, hq, hkv, d, "f32", 1e4)
    c = torch.tensor(ctx, dtype=torch.int32, device=DEV)
    out = torch.full((B, n, hq, d), 7.0, device=DEV)
    if decode:
        pic.pic_decode_attn(model, t["q"], t["k"], t["v"], t["K"], t["V"], B, cap, c, 0, max(ctx), out)
    else:
        pic.pic_suffix_prefill_attn(model, t["q"], t["k"], t["v"], t["K"], t["V"], B, cap, c, max(ctx), n, out)
    torch.cuda.synchronize()
    return h, out.cpu().numpy(), t["K"].cpu().numpy(), t["V"].cpu().numpy()


def _check(h, out, K, V, ctx):
    for b, c in enumerate(ctx):
        ref, K2, V2 = O.suffix_prefill(h["K"][b][:, :c], h["V"][b][:, :c], h["q"][b], h["k"][b], h["v"][b])
        assert np.abs(out[b] - ref).max() <= 1e-5
        n = c + h["q"].shape[1]
        assert np.array_equal(K[b][:, :n], K2.astype(np.float32)) and np.array_equal(V[b][:, :n], V2.astype(np.float32))
        assert np.array_equal(K[b][:, n:], h["K"][b][:, n:]) and np.array_equal(V[b][:, n:], h["V"][b][:, n:])


# (query heads, kv heads, head_dim, context lengths, suffix tokens)
SHAPES = [
    (4, 2, 64, [0], 1), (4, 2, 64, [1, 15, 16, 17], 3), (4, 2, 64, [127, 128, 129, 300], 16),
    (4, 2, 128, [0, 1, 16], 17), (3, 1, 64, [33, 200], 11), (5, 1, 128, [40, 64], 7), (2, 2, 128, [255, 31], 33),
    (16, 4, 64, [97] * 20, 61),     # 80 pairs x 8 m-tiles of 32 rows: the 32-row workgroups
    (16, 4, 128, [65, 97, 0, 143] * 5, 64),
]


@pytest.mark.parametrize("hq,hkv,d,ctx,n_q", SHAPES)
def test_prefill_edges(hq, hkv, d, ctx, n_q):
    _check(*_run(hq, hkv, d, ctx, n_q), ctx)


@pytest.mark.parametrize("hq,hkv,d,ctx", [(4, 2, 64, [0, 1, 15, 16, 127, 128, 400]), (40, 2, 128, [16, 31, 250]),
                                          (16, 4, 64, [70] * 70)])
def test_decode_edges(hq, hkv, d, ctx):
    _check(*_run(hq, hkv, d, ctx, None), ctx)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("d,batch", [(64, 1), (128, 1), (64, 40)])
def test_a_value_that_is_not_finite_reaches_only_the_rows_that_see_it(d, batch, bad):
    ctx, n_q, at = [45] * batch, 20, 9

    def plant(h):
        h["v"][:, at, :, 3] = bad

    clean = _run(16, 4, d, ctx, n_q)[1]
    out = _run(16, 4, d, ctx, n_q, plant=plant)[1]
    assert np.array_equal(out[:, :at], clean[:, :at])          # earlier tokens: bit for bit
    assert np.array_equal(np.delete(out, 3, -1), np.delete(clean, 3, -1))
    assert not np.isfinite(out[:, at:, :, 3]).any()
    # past the last visible slot nothing is read into the sums
    def past(h):
        h["K"][:, :, max(ctx) + n_q:] = bad
        h["V"][:, :, max(ctx) + n_q:] = bad
    assert np.array_equal(_run(16, 4, d, ctx, n_q, plant=past)[1], clean)
