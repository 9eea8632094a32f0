"""Slot and tile maps at the sizes where their launch changes: one span, several, the last one partial,
many spans, and block lists long enough for the three separate launches; against the host's expansion."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2607_28069_amd as pic  # noqa: E402


@pytest.mark.parametrize("batch,cap,n_blocks", [(1, 1, 0), (1, 63, 1), (2, 64, 3), (1, 1024, 16), (3, 1025, 60), (2, 5000, 150),
                                                (40, 8200, 3000),          # 360 spans
                                                (64, 16384, 40000)])       # the separate launches
@pytest.mark.parametrize("tiles", [True, False])
def test_maps(batch, cap, n_blocks, tiles):
    rng = np.random.default_rng(batch * cap + n_blocks)
    blocks = np.zeros(max(n_blocks, 1), pic.BLOCK_DTYPE)
    # aligned runs, shifted ones, gaps, one-token and invalid blocks; no slot covered twice
    slots = [(b, s) for b in range(batch) for s in range(0, cap, 64)]
    order = rng.permutation(len(slots))
    n = 0
    for j in order[:n_blocks]:
        b, s = slots[j]
        k = int(rng.integers(1, 65)) if rng.random() < 0.4 else 64
        blocks[n] = (b, int(rng.integers(0, 1 << 20)) if rng.random() < 0.5 else 64 * s, s, min(k, cap - s), int(rng.integers(-99, 99)))
        n += 1
    while n < n_blocks:   # the rest: out of range, skipped
        blocks[n] = [(batch, 0, 0, 1, 0), (0, 0, cap, 1, 0), (0, 0, -1, 1, 0), (0, 0, 0, 65, 0), (-1, 0, 0, 64, 0)][n % 5]
        n += 1
    src, dl = np.zeros((batch, cap), np.int32), np.zeros((batch, cap), np.int32)
    for b, t, s, k, d in blocks[:n_blocks].tolist():
        if 0 <= b < batch and 0 < k <= 64 and s >= 0 and s + k <= cap:
            src[b, s:s + k] = t + np.arange(k)
            dl[b, s:s + k] = d
    nt = pic.pic_slot_map_tiles(cap)
    want = np.zeros((batch, nt, 2), np.int32)
    want[:, :, 0] = -1
    for b in range(batch):
        for t in range(cap // 64):
            x, y = src[b, 64 * t:64 * t + 64], dl[b, 64 * t:64 * t + 64]
            if (x == x[0] + np.arange(64)).all() and (y == y[0]).all():
                want[b, t] = x[0], y[0]
    dev = torch.from_numpy(blocks.view(np.int32).copy()).cuda()
    a, c = (torch.full((batch, cap), 123, dtype=torch.int32, device="cuda") for _ in range(2))
    tm = torch.full((batch, nt, 2), 123, dtype=torch.int32, device="cuda") if tiles else None
    pic.pic_build_slot_map(dev, n_blocks, batch, cap, a, c, tm)
    torch.cuda.synchronize()
    assert np.array_equal(a.cpu().numpy(), src) and np.array_equal(c.cpu().numpy(), dl)
    if tiles:
        assert np.array_equal(tm.cpu().numpy(), want)


def test_the_largest_map():
    """map_cap of 2^31 - 1 slots: blocks at both ends and in the last 4096 slots."""
    cap = 2 ** 31 - 1
    rows = [(0, 5, 0, 64, 7), (0, 100, cap - 64, 64, -9), (0, 300, cap - 4000, 50, 3), (0, 400, 2 ** 30, 64, 1)]
    blocks = torch.tensor(rows, dtype=torch.int32, device="cuda")
    src, dl = (torch.full((cap,), -5, dtype=torch.int32, device="cuda") for _ in range(2))
    tiles = torch.full((2 ** 25, 2), -5, dtype=torch.int32, device="cuda")
    pic.pic_build_slot_map(blocks, len(rows), 1, cap, src, dl, tiles)
    torch.cuda.synchronize()
    for _, s, d, n, shift in rows:
        assert torch.equal(src[d:d + n], torch.arange(s, s + n, dtype=torch.int32, device="cuda"))
        assert bool((dl[d:d + n] == shift).all())
    covered = sum(n for _, _, _, n, _ in rows)
    # (counted in pieces: a mask of the whole map at once would be another 2 GB)
    assert sum(int(torch.count_nonzero(p)) for p in dl.split(1 << 28)) == covered
    whole = torch.nonzero(tiles[:, 0] >= 0).flatten().tolist()
    assert whole == [0, 2 ** 24]
    assert tiles[0].tolist() == [5, 7] and tiles[2 ** 24].tolist() == [400, 1] and tiles[-1].tolist() == [-1, 0]


# lists of short blocks (their finder expands up to 8 tokens), at the limits of the one-launch form: 512 spans,
# 8192 blocks
@pytest.mark.parametrize("batch,cap,lens", [(3, 2500, range(1, 13)), (1, 8192, [1]), (1, 8193, [1]), (512, 1000, [64, 9]),
                                            (513, 1000, [64, 9]), (2, 4000, [8, 9])])
def test_short_blocks(batch, cap, lens):
    rows, k = [], 0
    for b in range(batch):
        p = 0
        while p < cap:
            n = min(lens[k % len(lens)], cap - p)
            rows.append((b, 7 * k % 5000, p, n, k % 11 - 5))
            p, k = p + n, k + 1
    _maps_equal_host(rows, batch, cap)


def test_more_blocks_in_a_span_than_its_list_holds():
    rows = [(0, 100, 64, 64, 3)] * 300 + [(0, 9, 1000, 50, -2)] * 5   # (the same run many times)
    _maps_equal_host(rows, 2, 2000)


def _maps_equal_host(rows, batch, cap):
    r = np.asarray(rows, np.int32)
    src, dl = np.zeros((batch, cap), np.int32), np.zeros((batch, cap), np.int32)
    for b, t, s, k, d in rows:
        src[b, s:s + k] = t + np.arange(k)
        dl[b, s:s + k] = d
    nt = pic.pic_slot_map_tiles(cap)
    a, c = (torch.full((batch, cap), 123, dtype=torch.int32, device="cuda") for _ in range(2))
    tm = torch.full((batch, nt, 2), 123, dtype=torch.int32, device="cuda")
    pic.pic_build_slot_map(torch.from_numpy(r.copy()).cuda(), len(rows), batch, cap, a, c, tm)
    torch.cuda.synchronize()
    assert np.array_equal(a.cpu().numpy(), src) and np.array_equal(c.cpu().numpy(), dl)
    s64, d64 = src[:, :cap // 64 * 64].reshape(batch, -1, 64), dl[:, :cap // 64 * 64].reshape(batch, -1, 64)
    run = (s64 == s64[:, :, :1] + np.arange(64)).all(-1) & (d64 == d64[:, :, :1]).all(-1)
    want = np.zeros((batch, nt, 2), np.int32)
    want[:, :, 0] = -1
    want[:, :cap // 64][run] = np.stack([s64[:, :, 0], d64[:, :, 0]], -1)[run]
    assert np.array_equal(tm.cpu().numpy(), want)
