"""The TopK merge at the edges of its tiles, against numpy's sort: list lengths
around one and two 128-entry tiles and one 512-position fill workgroup, 1 to 17
lists (two and three rounds of eight), full, ragged and empty lists, and brackets
that do not fit in LDS (every priority equal, one list interleaving all others)."""
import numpy as np
import pytest
import torch

from paper_2310_05205_amd import gear
from tests.helpers import cuda, host, say

pytestmark = pytest.mark.gpu


def _lists(G, K, kind, rng):
    prio, gidx = np.zeros((G, K), np.uint32), np.full((G, K), -1, np.int64)
    for g in range(G):
        n = K if kind in ("full", "equal", "blocks") else 0 if kind == "empty" else int(rng.integers(0, K // G + 2))
        if kind == "one full" and g == G - 1:
            n = K
        n = min(n, K)
        slots = np.sort(rng.permutation(4 * K)[:n]) * G + g if kind != "blocks" else np.arange(n) + g * 4 * K
        p = np.full(n, 7) if kind == "equal" else rng.integers(1, 1 << 32 if kind == "full" else 50, n)
        order = np.lexsort((slots, -p))
        prio[g, :n], gidx[g, :n] = p[order], slots[order]
    return prio, gidx


@pytest.mark.parametrize("G,K", [(1, 1), (2, 127), (3, 128), (8, 129), (9, 511), (16, 513), (17, 1000), (8, 8192),
                                 (5, 16384)])
@pytest.mark.parametrize("kind", ["full", "ragged", "one full", "equal", "blocks", "empty"])
def test_merge_matches_sort(G, K, kind):
    say("G=%d K=%d %s" % (G, K, kind))
    rng = np.random.default_rng(G * 100003 + K)
    prio, gidx = _lists(G, K, kind, rng)
    flat_p, flat_i = prio.reshape(-1).astype(np.int64), gidx.reshape(-1)
    valid = np.flatnonzero(flat_i >= 0)
    best = valid[np.lexsort((flat_i[valid], -flat_p[valid]))][:K]
    want_i, want_p = np.full(K, -1, np.int64), np.zeros(K, np.int64)
    want_i[: best.size], want_p[: best.size] = flat_i[best], flat_p[best]
    idx, start, w, p = gear.topk_merge(torch.from_numpy(prio.view(np.int32)).to(cuda()),
                                       torch.from_numpy(gidx).to(cuda()), K, 9, 4, 3)
    np.testing.assert_array_equal(host(idx), want_i)
    np.testing.assert_array_equal(host(p).view(np.uint32), want_p)
    np.testing.assert_array_equal(host(w), (want_i >= 0).astype(np.float32))
    assert (host(start)[want_i < 0] == 0).all() and (host(start) >= 0).all() and (host(start) <= 5).all()
