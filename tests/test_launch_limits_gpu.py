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
