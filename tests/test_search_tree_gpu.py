"""Prioritized selection at the edges of its sum tree, against the oracle.

Table sizes on both sides of every change of layout: the one-launch limit
(16384), whole and ragged tiles (256) and chunks (4096 slots, 16384 above 2^22),
the highest level's two search rounds and three (256 nodes), chunks of 16 and 64
tiles (2^22) and two and three levels (2^24); batches below, at and above one
draw per 16-lane row of the largest grid (16384).  Updates follow each select,
so the kept tree and the rescanned one must both agree."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_05205_amd import gear
from tests.helpers import assert_weights, cuda, host, say

pytestmark = pytest.mark.gpu

SIZES = [(16385, 300), (20479, 17), (20480, 16), (20481, 15), (65536, 16384), (65537, 16385), (1048576, 4000),
         (1048577, 4001), (4194304, 1000), (4194305, 1000), (4210689, 40000), (16777216, 2049), (16777217, 2049),
         (16777216 + 16384 * 257 + 5, 3000)]


@pytest.mark.parametrize("options", [0, gear.GEAR_OPT_INCREMENTAL_TREE, gear.GEAR_OPT_IS_GLOBAL_MIN],
                         ids=["rescan", "incremental", "global-min"])
@pytest.mark.parametrize("N,B", SIZES)
def test_tree_edges(N, B, options):
    rng = np.random.default_rng(N)
    p = rng.integers(1, 1 << 20, N).astype(np.uint32)
    p[rng.random(N) < 0.3] = 0
    p[: N // 2 : 4096] = 0xFFFFFFFF  # sums beyond 32 bits in single tiles
    global_min = options == gear.GEAR_OPT_IS_GLOBAL_MIN
    p[p == 1] = 2
    # A draw of the last slot likely; or the table's only smallest priority there,
    # in the last chunk.
    p[-1] = 1 if global_min else 0xFFFFFFFF
    t = gear.Table([], N, 1)
    try:
        t.set_options(options)
        t.insert([], p)
        for it in range(2):
            say("N=%d B=%d options=%d iteration %d" % (N, B, options, it))
            idx, start, w = t.select(gear.GEAR_PRIORITIZED, B, 1, 77 + it, 0.4, weights=True)
            st, oidx, ostart, ow = oracle.select(3, p, N, 1, B, 1, 77 + it, 0.4, True, global_min=global_min)
            assert st == oracle.OK
            np.testing.assert_array_equal(host(idx), oidx)
            np.testing.assert_array_equal(host(start), ostart)
            assert_weights(host(w), ow)
            new = rng.integers(0, 1 << 20, B).astype(np.uint32)
            new[new == 1] = 2
            t.update_priorities(idx, torch.from_numpy(new.view(np.int32)).to(cuda()))
            oracle.update(p, oidx, new)
        np.testing.assert_array_equal(t.priorities(), p)
        assert t.sync() == 0
    finally:
        t.close()


def test_every_slot_of_a_small_tree_is_found():
    """Draws over a table of ones reach each slot: every lane and position of
    the row search, in whole and ragged tiles."""
    N = 16384 + 300
    t = gear.Table([], N, 1)
    try:
        p = np.ones(N, np.uint32)
        t.insert([], p)
        seen = np.zeros(N, np.int64)
        for s in range(8):
            idx, _, _ = t.select(gear.GEAR_PRIORITIZED, 40000, 1, s)
            st, oidx, _, _ = oracle.select(3, p, N, 1, 40000, 1, s, 0.0, False)
            assert st == oracle.OK
            np.testing.assert_array_equal(host(idx), oidx)
            seen += np.bincount(oidx, minlength=N)
        assert (seen > 0).all()
    finally:
        t.close()
