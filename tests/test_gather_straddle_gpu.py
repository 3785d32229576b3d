"""Gathers of windows that are not whole 16-byte elements, and of sources at
any byte, against torch indexing of the same rows.

An odd window is moved in 16-byte elements, some of which hold the end of one
window and the start of the next; the sizes here lie on both sides of each
rule of that path: windows of 15 to 17 bytes and around the smallest that a
piece can stage (33 bytes in 8 KiB pieces, 130 in 32 KiB ones), windows just
below, at and above a piece, batches whose last element is short, and batches
of at least 128 MiB.  Draws without a window (index -1) and invalid ones read
as zeros beside valid neighbours."""
import numpy as np
import pytest
import torch

from paper_2310_05205_amd import gear
from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu

# (bytes per step, T, L, B)
CASES = [(15, 4, 1, 7), (16, 4, 1, 300), (17, 4, 1, 5000), (11, 9, 3, 1000), (32, 3, 1, 1001), (33, 5, 1, 1001),
         (34, 5, 1, 4099), (7, 40, 13, 3001), (147, 75, 13, 3001), (147, 75, 1, 1), (68, 50, 20, 512), (6, 30, 9, 777),
         (8191, 3, 1, 33), (8193, 3, 1, 33), (4097, 5, 2, 40), (4096, 5, 2, 40), (2731, 7, 3, 41), (100003, 2, 1, 9),
         (129, 4, 1, 1100000), (130, 4, 1, 1050000), (131, 4, 1, 1030003), (32767, 2, 1, 4200), (32769, 2, 1, 4200)]


@pytest.mark.parametrize("E,T,L,B", CASES)
@pytest.mark.parametrize("holes", [False, True])
def test_odd_windows_match_indexing(E, T, L, B, holes):
    N = 37
    rng = np.random.default_rng(E * 1000 + L)
    t = gear.Table([E, 4], N, T)
    try:
        g = torch.Generator(device="cuda")
        g.manual_seed(E)
        rows = torch.randint(1, 256, (N, T * E), dtype=torch.uint8, device=cuda(), generator=g)
        tags = torch.randint(1, 256, (N, T * 4), dtype=torch.uint8, device=cuda(), generator=g)
        t.insert([rows, tags], np.ones(N, np.uint32))
        idx = rng.integers(0, N, B)
        start = rng.integers(0, T - L + 1, B).astype(np.int32)
        start[: B // 2 + 1] = T - L  # the last window of the last slot ends with the column
        idx[: B // 3 + 1] = N - 1
        good = np.ones(B, bool)
        if holes:
            idx[rng.random(B) < 0.2] = -1
            idx[B // 2] = N + 5
            good = (idx >= 0) & (idx < N)
        d_idx, d_start = torch.from_numpy(idx).to(cuda()), torch.from_numpy(start).to(cuda())
        raw, small = t.collect(d_idx, d_start, L)
        ok = torch.from_numpy(good).to(cuda())
        for out, src, e in ((raw, rows, E), (small, tags, 4)):
            for b0 in range(0, B, 1 << 16):  # 64 Ki windows at a time
                b1 = min(B, b0 + (1 << 16))
                first = (d_start[b0:b1].long() * e)[:, None] + torch.arange(L * e, device=cuda())
                i = torch.where(ok[b0:b1], d_idx[b0:b1], 0)[:, None]
                want = torch.where(ok[b0:b1, None], src[i, first], torch.zeros((), dtype=torch.uint8, device=cuda()))
                assert torch.equal(out[b0:b1], want), (b0, e)
        assert t.sync() == (gear.GEAR_STATUS_BAD_INDEX if holes else 0)
    finally:
        t.close()


@pytest.mark.parametrize("E,T,L,B", [(17, 40, 13, 900), (147, 75, 13, 700), (9000, 3, 2, 60)])
def test_odd_windows_of_a_pinned_table_and_of_fused_draws(E, T, L, B):
    rows = torch.randint(1, 256, (64, T * E), dtype=torch.uint8)
    both = []
    for residency in (gear.GEAR_DEVICE, gear.GEAR_HOST_PINNED):
        t = gear.Table([E], 64, T, residency=residency)
        try:
            t.insert([rows], np.ones(64, np.uint32))
            idx, start, _, out = t.select_collect(gear.GEAR_UNIFORM, B, L, 9)
            idx2, start2, _ = t.select(gear.GEAR_UNIFORM, B, L, 9)
            assert torch.equal(idx, idx2) and torch.equal(start, start2)
            assert torch.equal(out[0], t.collect(idx, start, L)[0])
            both.append((host(idx), host(start), host(out[0])))
            assert t.sync() == 0
        finally:
            t.close()
    for x, y in zip(*both):
        assert np.array_equal(x, y)
    idx, start, out = both[0]
    cols = start.astype(np.int64)[:, None] * E + np.arange(L * E)
    assert np.array_equal(out, rows.numpy()[idx[:, None], cols])
