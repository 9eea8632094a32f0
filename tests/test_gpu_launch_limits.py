"""Calls whose workgroups exceed what one grid dimension can launch (2^32 threads): batches of a million
one- or two-key requests."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_28069_amd as pic  # noqa: E402

DEV = "cuda"


def test_float32_decode_of_8_million_pairs():
    B, H, d = (1 << 20) + 1, 8, 64   # 2^23 + 8 workgroups of 512 threads
    m = pic.Model.of(1, H, H, d, "f32", 5e5)
    q, k, v = (torch.randn((B, H, d), device=DEV) for _ in range(3))
    K, V, out = (torch.full((B, H, d), float("nan"), device=DEV) for _ in range(3))
    pic.pic_decode_attn(m, q, k, v, K, V, B, 1, torch.zeros(B, dtype=torch.int32, device=DEV), 0, 0, out, None)
    torch.cuda.synchronize()
    assert torch.equal(K, k) and torch.equal(V, v)
    # one key: p v / p, two float32 roundings of 2^-24 each
    assert bool(((out - v).abs() <= 2.0 ** -22 * v.abs()).all())


def test_split_decode_of_16_million_query_rows():
    B, hq, d = (1 << 20) + 1, 16, 64   # 2^24 + 16 rows, 256 threads each, to combine
    m = pic.Model.of(1, hq, 1, d, "bf16", 5e5)
    f = lambda *s: torch.randn(s, device=DEV, dtype=torch.bfloat16)
    q, k, v, K, V = f(B, hq, d), f(B, 1, d), f(B, 1, d), f(B, 1, 2, d), f(B, 1, 2, d)
    out = torch.full_like(q, float("nan"))
    ws = torch.empty(pic.pic_decode_workspace_bytes(m, B, 2, 2), dtype=torch.uint8, device=DEV)
    pic.pic_decode_attn(m, q, k, v, K, V, B, 2, torch.ones(B, dtype=torch.int32, device=DEV), 0, 1, out, ws, n_splits=2)
    torch.cuda.synchronize()
    assert torch.equal(K[:, :, 1], k) and torch.equal(V[:, :, 1], v)
    for b0 in range(0, B, 1 << 16):   # two keys: a weight and its complement
        s = slice(b0, b0 + (1 << 16))
        K32, V32 = K[s, 0].float(), V[s, 0].float()
        w = torch.sigmoid((q[s].float() * (K32[:, 0] - K32[:, 1])[:, None]).sum(-1, keepdim=True) / d ** 0.5)
        ref = w * V32[:, None, 0] + (1 - w) * V32[:, None, 1]
        assert bool(((out[s].float() - ref).abs() <= 2e-2 + 1e-2 * ref.abs()).all()), b0
