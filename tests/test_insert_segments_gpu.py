"""Insertion from device memory in one launch, against rows written by numpy.

Row sizes that are and are not multiples of 16 bytes, sources and slots at odd
addresses, batches that wrap the ring or exceed it, priorities in pageable,
page-locked and device memory, more columns than one launch takes, and slot lists
of the index manager as one run, several, descending and scattered."""
from collections import deque

import numpy as np
import pytest
import torch

from paper_2310_05205_amd import gear
from tests.helpers import cuda, host, say

pytestmark = pytest.mark.gpu


def _rows(n, row, shift, rng):
    """n rows of `row` bytes on the GPU, `shift` bytes past an aligned address."""
    data = rng.integers(0, 256, n * row, dtype=np.uint8)
    buf = torch.zeros(n * row + 16, dtype=torch.uint8, device=cuda())
    buf[shift:shift + n * row] = torch.from_numpy(data).to(cuda())
    return data.reshape(n, row), buf[shift:shift + n * row].view(n, row)


def _priorities(p, kind):
    if kind == "pageable":
        return p
    t = torch.from_numpy(p.view(np.int32))
    return t.pin_memory() if kind == "pinned" else t.to(cuda())


def _check(t, model, prio):
    for c, want in enumerate(model):
        np.testing.assert_array_equal(host(t.column_view(c)), want)
    np.testing.assert_array_equal(t.priorities(), prio)


@pytest.mark.parametrize("kind", ["pageable", "pinned", "device"])
@pytest.mark.parametrize("cols,T,N", [([16], 4, 9), ([1, 3, 68], 5, 37), ([7, 2, 12288], 3, 11), ([1] * 45, 1, 700),
                                      ([1023, 1025], 1, 6)])
def test_ring_insert(cols, T, N, kind):
    rng = np.random.default_rng(len(cols) * N)
    t = gear.Table(cols, N, T)
    try:
        model = [np.zeros((N, T * e), np.uint8) for e in cols]
        prio, seq = np.zeros(N, np.uint32), 0
        for step, n in enumerate([1, N // 2, 3, N, 2, N + 5, 2 * N + 1, 7, 513, 512]):
            say("%s step %d n=%d" % (cols[:3], step, n))
            made = [_rows(n, T * e, (step * 5 + c) % 16, rng) for c, e in enumerate(cols)]
            p = rng.integers(1, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
            t.insert([d for _, d in made], _priorities(p, kind))
            for k in range(n):
                slot = (seq + k) % N
                for m, (h, _) in zip(model, made):
                    m[slot] = h[k]
                prio[slot] = p[k]
            seq += n
            _check(t, model, prio)
        assert t.sync() == 0
    finally:
        t.close()


def _runs(slots):
    """Runs of consecutive slots, ascending or descending, in a list of victims."""
    runs, k = 0, 0
    while k < len(slots):
        step = -1 if k + 1 < len(slots) and slots[k + 1] == slots[k] - 1 else 1
        k += 1
        while k < len(slots) and slots[k] == slots[k - 1] + step:
            k += 1
        runs += 1
    return runs


@pytest.mark.parametrize("removal", [gear.GEAR_FIFO, gear.GEAR_LIFO])
def test_managed_insert(removal):
    """The victims are named by the commit order that the test keeps itself:
    the oldest under FIFO, the newest under LIFO, in lists of every number of runs
    that travels in a kernel's arguments and of more."""
    cols, T, N = [5, 64, 33], 3, 40
    rng = np.random.default_rng(int(removal))
    t = gear.Table(cols, N, T)
    try:
        t.use_allocator(removal)
        model = [np.zeros((N, T * e), np.uint8) for e in cols]
        prio = np.zeros(N, np.uint32)
        order, seen = deque(), set()
        for step in range(60):
            n = int(rng.integers(1, 30))
            idx = t.allocate(n)
            victims = [order.popleft() if removal == gear.GEAR_FIFO else order.pop()
                       for _ in range(max(0, len(order) + n - N))]
            seen.add(min(_runs(victims), 9))
            prio[victims] = 0
            perm = rng.permutation(n) if step % 3 == 0 else np.arange(n)[::-1] if step % 3 == 1 else np.arange(n)
            idx = np.ascontiguousarray(idx[perm])
            made = [_rows(n, T * e, step % 16, rng) for e in cols]
            p = rng.integers(1, 1000, n).astype(np.uint32)
            np.testing.assert_array_equal(t.priorities(), prio)  # the victims and no other slot
            t.write_rows(idx, [d for _, d in made])
            t.commit(idx, _priorities(p, ("pageable", "pinned", "device")[step % 3]))
            for m, (h, _) in zip(model, made):
                m[idx] = h
            prio[idx] = p
            order.extend(idx.tolist())
            assert t.allocator_info() == (len(order), 0, N - len(order))
            np.testing.assert_array_equal(t.priorities(), prio)
            for c, want in enumerate(model):
                np.testing.assert_array_equal(host(t.column_view(c)), want)
        assert {0, 1, 8, 9} <= seen
        assert t.sync() == 0
    finally:
        t.close()


def test_columns_on_the_host_or_mixed_take_the_copies():
    t = gear.Table([8, 8], 10, 2)
    try:
        a = torch.arange(160, dtype=torch.uint8).reshape(10, 16)
        b = (a + 1).to(cuda())
        t.insert([a.pin_memory(), b], np.arange(1, 11, dtype=np.uint32))
        torch.cuda.synchronize()
        np.testing.assert_array_equal(host(t.column_view(0)), a.numpy())
        np.testing.assert_array_equal(host(t.column_view(1)), host(b))
        t.insert([a[:4].numpy().copy(), b[:4]], np.full(4, 9, np.uint32))
        np.testing.assert_array_equal(t.priorities(), [9, 9, 9, 9, 5, 6, 7, 8, 9, 10])
    finally:
        t.close()


def test_rows_of_the_table_itself_keep_the_order_of_the_copies():
    """Sources in the table's own columns and priorities, not next to their
    destinations: the first part of a wrapped batch is written before the second,
    and a column before the next one."""
    N, E = 4096, 64
    rng = np.random.default_rng(3)
    t = gear.Table([E, E], N, 1)
    try:
        rows = [rng.integers(0, 256, (N, E), dtype=np.uint8) for _ in range(2)]
        p = rng.integers(1, 1000, N).astype(np.uint32)
        t.insert(rows, p)
        t.insert([r[:N - 1000] for r in rows], p[:N - 1000])  # the next batch wraps after 1000 rows
        n = 2000
        views = [t.column_view(c).view(N, E)[:n] for c in range(2)]
        t.insert(views, np.full(n, 5, np.uint32))
        for m in rows:
            m[N - 1000:] = m[:1000].copy()
            m[:1000] = m[1000:2000].copy()
        for c in range(2):
            np.testing.assert_array_equal(host(t.column_view(c)).reshape(N, E), rows[c])
    finally:
        t.close()


def test_managed_rows_of_another_column():
    """Column 1 takes the rows that the same call has written to column 0."""
    N, E = 4096, 64
    rng = np.random.default_rng(4)
    t = gear.Table([E, E], N, 1)
    try:
        t.use_allocator(gear.GEAR_FIFO)
        idx = t.allocate(N)
        new = rng.integers(0, 256, (N, E), dtype=np.uint8)
        t.write_rows(idx, [torch.from_numpy(new).to(cuda()), t.column_view(0)])
        got = [host(t.column_view(c)).reshape(N, E) for c in range(2)]
        np.testing.assert_array_equal(got[0][idx], new)
        np.testing.assert_array_equal(got[1][idx], got[0])
    finally:
        t.close()
