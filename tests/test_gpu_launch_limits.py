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
