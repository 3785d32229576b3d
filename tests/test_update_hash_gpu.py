"""Priority updates at the edges of the one-launch kernels, against the oracle.

Batches around one draw, a wave, each kernel's largest batch (1024, 2048, 4096,
8192) and the first two-launch one, over index patterns that stress the hash
tables: one slot for the whole batch, every slot twice, distinct slots, strides,
and slots of a single partition (multiples of the partition hash's inverse, so
that one workgroup receives every draw and its table fills to half)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_05205_amd import gear
from tests.helpers import cuda, host, say

pytestmark = pytest.mark.gpu

N = 70001
BATCHES = [1, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193]
INVERSE = pow(0x85EBCA6B, -1, 1 << 32)


def _patterns(B, rng):
    yield "one slot", np.full(B, N - 1)
    yield "pairs", np.repeat(rng.permutation(N)[: (B + 1) // 2], 2)[:B]
    yield "distinct", rng.permutation(N)[:B]
    yield "random", rng.integers(0, N, B)
    yield "stride 8", np.arange(B) * 8 % N
    # Slots whose hash lies below 2^32 / 64: partition 0 of 32 and of 64.
    h = np.arange(N, dtype=np.uint64) * np.uint64(0x85EBCA6B) & np.uint64(0xFFFFFFFF)
    slots = np.flatnonzero(h < (1 << 26))
    assert INVERSE * 0x85EBCA6B % (1 << 32) == 1 and slots.size > 500
    yield "one partition", rng.choice(slots, B)


@pytest.mark.parametrize("options", [0, gear.GEAR_OPT_INCREMENTAL_TREE], ids=["rescan", "incremental"])
@pytest.mark.parametrize("B", BATCHES)
def test_update_patterns(B, options):
    rng = np.random.default_rng(B)
    p = rng.integers(0, 1 << 20, N).astype(np.uint32)
    t = gear.Table([], N, 1)
    try:
        t.set_options(options)
        t.insert([], p)
        for name, idx in _patterns(B, rng):
            say("B=%d %s" % (B, name))
            t.select(gear.GEAR_PRIORITIZED, 3000, 1, 1)  # the kept tree is current before the update
            new = rng.integers(0, 1 << 32, B, dtype=np.uint64).astype(np.uint32)
            t.update_priorities(torch.from_numpy(idx.astype(np.int64)).to(cuda()),
                                torch.from_numpy(new.view(np.int32)).to(cuda()))
            oracle.update(p, idx, new)
            np.testing.assert_array_equal(t.priorities(), p, err_msg=name)
            got, _, _ = t.select(gear.GEAR_PRIORITIZED, 3000, 1, B)
            st, want, _, _ = oracle.select(3, p, N, 1, 3000, 1, B, 0.0, False)
            assert st == oracle.OK
            np.testing.assert_array_equal(host(got), want, err_msg=name)
        assert t.sync() == 0
    finally:
        t.close()


@pytest.mark.parametrize("B", [1, 1000, 3000, 8192])
def test_invalid_indices_are_reported_and_skipped(B):
    p = np.arange(1, N + 1, dtype=np.uint32)
    t = gear.Table([], N, 1)
    try:
        t.insert([], p)
        idx = np.random.default_rng(B).integers(0, N, B)
        idx[B - 1] = N
        new = np.full(B, 7, np.int32)
        t.update_priorities(torch.from_numpy(idx).to(cuda()), torch.from_numpy(new).to(cuda()))
        assert t.sync() == gear.GEAR_STATUS_BAD_INDEX
        p[idx[idx < N]] = 7
        np.testing.assert_array_equal(t.priorities(), p)
    finally:
        t.close()
