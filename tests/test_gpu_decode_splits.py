"""Split decode of requests of uneven lengths, where the key ranges are dealt by length, and the split
counts the launch picks by itself, with and without a workspace.

Reference: float64 attention on the device over the same bf16 values; tolerance: the bf16 bar of the
parity tests (2e-2 absolute + 1e-2 relative, 1e-2 in the 2-norm)."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_28069_amd as pic  # noqa: E402

DEV = "cuda"


def _inputs(hq, hkv, d, base, step, seed=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    f = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16)
    B, cap = len(base), max(base) + step + 1
    return dict(model=pic.Model.of(1, hq, hkv, d, "bf16", 5e5), q=f(B, hq, d), k=f(B, hkv, d), v=f(B, hkv, d),
                K=f(B, hkv, cap, d), V=f(B, hkv, cap, d), base=torch.tensor(base, dtype=torch.int32, device=DEV),
                out=torch.full((B, hq, d), float("nan"), device=DEV, dtype=torch.bfloat16), B=B, cap=cap)


def _decode(x, base, step, n_splits, ws="query"):
    if ws == "query":
        n = pic.pic_decode_workspace_bytes(x["model"], x["B"], x["cap"], n_splits)
        ws = torch.full((max(n, 16) // 4,), float("nan"), device=DEV)
    pic.pic_decode_attn(x["model"], x["q"], x["k"], x["v"], x["K"], x["V"], x["B"], x["cap"], x["base"], step,
                        max(base), x["out"], ws, n_splits=n_splits)
    torch.cuda.synchronize()


def _check(x, base, step):
    for b, n in enumerate(base):
        p = n + step
        assert torch.equal(x["K"][b, :, p], x["k"][b]) and torch.equal(x["V"][b, :, p], x["v"][b])
        K, V = x["K"][b, :, :p + 1].double(), x["V"][b, :, :p + 1].double()
        hq, d = x["q"].shape[1:]
        q = x["q"][b].double().view(K.shape[0], -1, d)
        ref = torch.stack([torch.softmax(q[h] @ K[h].t().contiguous() / math.sqrt(d), -1) @ V[h]
                           for h in range(K.shape[0])]).view(hq, d)
        got = x["out"][b].double()
        assert bool(((got - ref).abs() <= 2e-2 + 1e-2 * ref.abs()).all()), (b, n)
        assert float((got - ref).norm() / ref.norm()) <= 1e-2, (b, n)


# lengths at and around the 128-key units and the 8192-key line, from one key to the longest
@pytest.mark.parametrize("hq,hkv,d,base,step,n_splits", [
    (8, 2, 128, [8192, 0, 1, 127, 128, 129, 5000], 0, 8),
    (8, 2, 128, [9000, 9000, 9000], 3, 8),                       # one length
    (8, 2, 64, [12345, 300, 8191, 64], 2, 13),
    (28, 4, 128, [20000, 10001], 1, 0),                          # as picked: 32 ranges on average
    (40, 1, 128, [8200, 37, 4100], 0, 9),                        # three groups of query heads
    (4, 1, 64, [8191 + i * 37 % 4000 for i in range(64)], 0, 8),  # as many requests as are dealt
    (4, 1, 64, [8300 - i for i in range(65)], 0, 8),             # one more: equal ranges
    (8, 2, 128, [8190, 2], 0, 8),                                # below the line: equal ranges
])
def test_uneven_lengths(hq, hkv, d, base, step, n_splits):
    x = _inputs(hq, hkv, d, base, step)
    _decode(x, base, step, n_splits)
    _check(x, base, step)


@pytest.mark.parametrize("batch", [20, 32, 33, 64])
def test_a_batch_that_fills_the_gpu_needs_no_workspace(batch):
    base = [4096 - 17 * b for b in range(batch)]
    x = _inputs(16, 8, 128, base, 0)
    splits = pic.pic_decode_auto_splits(x["model"], batch, x["cap"])
    assert splits == (4 if batch == 33 else 1)
    _decode(x, base, 0, 0)
    _check(x, base, 0)
    x["out"].fill_(float("nan"))
    if batch * 8 >= 256:
        _decode(x, base, 0, 0, ws=None)
        _check(x, base, 0)
        x["out"].fill_(float("nan"))
        pic.pic_decode_attn_noalloc(x["model"], x["q"], x["k"], x["v"], x["K"], x["V"], batch, x["cap"], x["base"], 0,
                                    max(base), x["out"])
        torch.cuda.synchronize()
        _check(x, base, 0)


def test_noalloc_full_launch_equals_the_call_without_a_workspace():
    base = [4200 - 17 * b for b in range(33)]
    outs = []
    for noalloc in (False, True):
        x = _inputs(16, 8, 128, base, 0)
        if noalloc:
            pic.pic_decode_attn_noalloc(x["model"], x["q"], x["k"], x["v"], x["K"], x["V"], 33, x["cap"], x["base"], 0,
                                        max(base), x["out"])
            torch.cuda.synchronize()
        else:
            _decode(x, base, 0, 0, ws=None)
        _check(x, base, 0)
        outs.append(x["out"])
    assert torch.equal(outs[0], outs[1])


# lengths against the greatest the call allows, whose equal ranges the host works out: all at it, all
# one unit or far below it, one below it, garbage above it (clamped)
@pytest.mark.parametrize("base,max_base", [([9000] * 3, 9000), ([9000] * 3, 9500), ([8300] * 3, 20000), ([9000, 9000, 8871], 9000),
                                           ([9000, 8999, 9000], 9000), ([30000, 12000, 9000], 9000)])
@pytest.mark.parametrize("d,n_splits", [(128, 8), (64, 40)])
def test_lengths_and_the_greatest_allowed(base, max_base, d, n_splits):
    x = _inputs(8, 2, d, [max_base] * len(base), 1)
    x["base"] = torch.tensor(base, dtype=torch.int32, device=DEV)
    ws = torch.full((pic.pic_decode_workspace_bytes(x["model"], 3, max_base + 2, n_splits) // 4,), float("nan"), device=DEV)
    pic.pic_decode_attn(x["model"], x["q"], x["k"], x["v"], x["K"], x["V"], 3, x["cap"], x["base"], 1, max_base, x["out"], ws,
                        n_splits=n_splits)
    torch.cuda.synchronize()
    _check(x, [min(b, max_base) for b in base], 1)
