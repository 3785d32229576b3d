"""TopK at the edges of its list, its early stops and its ranking, against the
oracle: K around a wave's four keys, a workgroup's 32 and a 256-entry chunk, a
whole bin taken beyond K (distinct values that share their leading bits), the
largest such bin and the first too large, ties across chunks, and every pass."""
import numpy as np
import pytest

import oracle
from paper_2310_05205_amd import gear
from tests.helpers import host, say

pytestmark = pytest.mark.gpu

KS = [1, 3, 4, 5, 31, 32, 33, 255, 256, 257, 511, 1000, 4096, 8191, 16384]


def _priorities(kind, N, rng):
    if kind == "distinct":  # any bin is small: the first pass decides with a bin taken whole
        return rng.permutation(1 << 24)[:N].astype(np.uint32) + (1 << 24)
    if kind == "narrow":    # one leading-digit bin holds everything: later passes decide
        return (np.uint32(1 << 31) + rng.permutation(N).astype(np.uint32))
    if kind == "ties":
        return rng.integers(1, 40, N).astype(np.uint32)
    if kind == "two bins":  # the first bin at the top is just below or above what may be ranked whole
        p = rng.integers(1, 256, N).astype(np.uint32)
        p[: N // 3] = (1 << 20) + rng.integers(0, 1 << 13, N // 3)
        return rng.permutation(p)
    p = rng.integers(0, 1 << 32, N, dtype=np.uint64).astype(np.uint32)
    p[rng.random(N) < 0.9] = 0  # few candidates: K may exceed them
    return p


@pytest.mark.parametrize("kind", ["distinct", "narrow", "ties", "two bins", "sparse"])
@pytest.mark.parametrize("N", [17, 4096, 16383, 16384, 16385, 20001, 70000])
def test_topk_edges(N, kind):
    rng = np.random.default_rng(N)
    p = _priorities(kind, N, rng)
    t = gear.Table([], N, 1)
    try:
        t.insert([], p)
        candidates = int((p != 0).sum())
        if candidates == 0:
            return
        for K in KS + [min(candidates, 16384), min(candidates + 1, 16384)]:
            say("N=%d %s K=%d" % (N, kind, K))
            idx, start, w = t.select(gear.GEAR_TOPK, K, 1, K, weights=True)
            st, oidx, ostart, ow = oracle.select(4, p, N, 1, K, 1, K, 0.0, True)
            assert st == (oracle.NO_WEIGHT if K > candidates else oracle.OK)
            np.testing.assert_array_equal(host(idx), oidx)
            np.testing.assert_array_equal(host(start), ostart)
            np.testing.assert_array_equal(host(w), ow)
            assert t.sync() == (gear.GEAR_STATUS_NO_WEIGHT if K > candidates else 0)
    finally:
        t.close()


@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_a_bin_at_the_limit_of_whole_ranking(extra):
    """K keys of which all but one lie above a bin whose size puts the list at
    its limit of K + K/4 + 256, one below and one above it."""
    K = 400
    bin_size = K + K // 4 + 256 - (K - 1) + extra
    rng = np.random.default_rng(3)
    p = np.concatenate([(1 << 28) + rng.permutation(1 << 18)[: K - 1], (1 << 20) + rng.permutation(1 << 13)[:bin_size],
                        rng.integers(1, 1000, 5000)]).astype(np.uint32)
    p = rng.permutation(p)
    t = gear.Table([], p.size, 1)
    try:
        t.insert([], p)
        idx, _, _ = t.select(gear.GEAR_TOPK, K, 1, 1)
        st, oidx, _, _ = oracle.select(4, p, p.size, 1, K, 1, 1, 0.0, False)
        assert st == oracle.OK
        np.testing.assert_array_equal(host(idx), oidx)
        assert t.sync() == 0
    finally:
        t.close()
