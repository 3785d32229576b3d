"""Calls cut into several launches give what one launch gives.

GEAR_TEST_MAX_WORK_ITEMS lowers a new table's limit of work items per launch (in
earnest 2^32, which no small call reaches)."""
import numpy as np
import pytest
import torch

from paper_2310_05205_amd import gear
from tests.helpers import cuda, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture
def limited(monkeypatch):
    """A table whose launches have at most 16384 work items: 256 KiB of rows."""
    tables = []

    def make(*args):
        monkeypatch.setenv("GEAR_TEST_MAX_WORK_ITEMS", "16384")
        tables.append(gear.Table(*args))
        monkeypatch.delenv("GEAR_TEST_MAX_WORK_ITEMS")
        return tables[-1]

    yield make
    for t in tables:
        t.close()


@pytest.mark.parametrize("how", ["ring", "managed", "scattered"])
@pytest.mark.parametrize("cols", [[3001, 16, 4], [70000, 5], [700001]])
def test_insertion(limited, cols, how):
    N, n = 23, 17
    rng = np.random.default_rng(cols[0])
    t = limited(cols, N, 1)
    if how == "managed":
        t.use_allocator(gear.GEAR_FIFO)
    model, prio = [np.zeros((N, e), np.uint8) for e in cols], np.zeros(N, np.uint32)
    for step in range(4):
        say("%s %s step %d" % (how, cols, step))
        slots = (step * n + np.arange(n)) % N
        if how == "scattered":
            slots = rng.permutation(N)[:n].astype(np.int64)
        rows = [rng.integers(0, 256, (n, e), dtype=np.uint8) for e in cols]
        p = rng.integers(1, 1000, n).astype(np.uint32)
        data = [torch.from_numpy(r).to(cuda()) for r in rows]
        if how == "scattered":
            t.write_rows(slots, data)
        else:
            t.insert(data, p)
            prio[slots] = p
        for m, r in zip(model, rows):
            m[slots] = r
        for c, m in enumerate(model):
            np.testing.assert_array_equal(host(t.column_view(c)), m)
        np.testing.assert_array_equal(t.priorities(), prio)
    assert t.sync() == 0


@pytest.mark.parametrize("residency", [gear.GEAR_DEVICE, gear.GEAR_HOST_PINNED])
@pytest.mark.parametrize("cols,T,B,L", [([1024, 32, 4], 40, 300, 32), ([147, 1, 2, 1], 30, 3001, 13),
                                        ([20000], 12, 40, 12), ([3, 16, 4] * 7, 25, 500, 9)])
def test_gather(limited, cols, T, B, L, residency):
    """Batches of several 64-workgroup launches, wide, narrow and straddling
    columns, against indexing; with a missing draw and the selection inside."""
    N = 60
    rng = np.random.default_rng(B)
    t = limited(cols, N, T, residency)
    rows = [rng.integers(0, 256, (N, T, e), dtype=np.uint8) for e in cols]
    t.insert([r.reshape(N, -1) for r in rows], np.ones(N, np.uint32))
    say("%s B=%d L=%d residency %d" % (cols[:4], B, L, residency))
    idx = rng.integers(0, N, B)
    start = rng.integers(0, T - L + 1, B).astype(np.int32)
    idx[B // 2] = -1
    got = t.collect(torch.from_numpy(idx).to(cuda()), torch.from_numpy(start).to(cuda()), L)
    fidx, fstart, _, fused = t.select_collect(gear.GEAR_UNIFORM, B, L, 7)
    sidx, sstart, _ = t.select(gear.GEAR_UNIFORM, B, L, 7)
    assert torch.equal(fidx, sidx) and torch.equal(fstart, sstart)
    fidx, fstart = host(fidx), host(fstart)
    steps = np.arange(L)
    for c, e in enumerate(cols):
        want = rows[c][idx[:, None], start[:, None] + steps].reshape(B, -1)
        want[B // 2] = 0
        np.testing.assert_array_equal(host(got[c]), want)
        np.testing.assert_array_equal(host(fused[c]),
                                      rows[c][fidx[:, None], fstart[:, None] + steps].reshape(B, -1))
    assert t.sync() == 0
