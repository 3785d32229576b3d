"""Calls larger than one launch may be, followed on the CPU.

The launch calls refuse 2^32 work items or more, which is 64 GiB of rows in the
copies and, in elements of 16 bytes, 128 GiB of a batch.  Every call here is larger,
or has a single row or window that is, and runs over a runtime that records
its launches: each must be allowed, and together they must copy every byte of
the call once, from where it lies to where it belongs."""
import ctypes

import numpy as np
import pytest

from tests import stub_runtime


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return stub_runtime.build(tmp_path_factory.mktemp("stub"))


def merged(copies):
    """Copies as maximal (dst, src, bytes), in order of the destination."""
    out = []
    for dst, src, n in sorted(copies):
        if out and out[-1][0] + out[-1][2] == dst and out[-1][1] + out[-1][2] == src:
            out[-1] = (out[-1][0], out[-1][1], out[-1][2] + n)
        else:
            out.append((dst, src, n))
    return out


def _scatter(name, args):
    """The (idx, src, dst, row bytes, rows' pieces, last piece's bytes, element bytes) of a row scatter."""
    at = [ctypes.cast(args[k], ctypes.POINTER(t)).contents.value for k, t in
          enumerate([ctypes.c_uint64] * 4 + [ctypes.c_uint32] * 2)]
    width = 16 if "IDv4_j" in name else 4 if "Ij" in name else 1
    return at[:3] + [at[3] * width, at[4], at[5] * width]


def insertion(rt, how, elem_bytes, N, T, before, n):
    """What a call of n rows copies and what it should, both merged."""
    gear, np_prio = rt.gear, np.ones(max(n, before), np.uint32)
    t = rt.table(elem_bytes, N, T)
    rb = [T * e for e in elem_bytes]
    src = [rt.device(n * r) for r in rb]
    if how == "managed":
        gear.gear_table_use_allocator(t, gear.GEAR_FIFO, N)
    if before:
        gear.gear_insert(t, before, src, np_prio.ctypes.data)
    del rt.launches[:], rt.copies[:]
    rt.reader = lambda name, args: (stub_runtime.read_segments(name, args) if "copy_segments" in name else
                                    _scatter(name, args) if "scatter_rows" in name else None)
    slots = (before + np.arange(n)) % N
    if how == "scattered":
        slots = slots[::-1].copy()
        gear.gear_write_rows(t, slots, src)
    else:
        gear.gear_insert(t, n, src, np_prio.ctypes.data)
    got, words = list(rt.copies), 0
    for l in rt.launches:
        name, grid, block, seen = l
        if "copy_segments" in name:
            got += stub_runtime.segment_copies(l)
            words += seen[2][1] if seen[2] else 0
        elif "scatter_rows" in name:
            idx, s, d, row, pieces, last = seen
            assert grid % pieces == 0 and (pieces - 1) * 1024 + last == row
            c = [k for k in range(len(rb)) if src[k] <= s < src[k] + n * rb[k]][0]
            first = (s - src[c]) // row
            got += [(d + int(slots[first + r]) * row, s + r * row, row) for r in range(grid // pieces)]
    want = [(rt.column(t, c) + int(slots[a]) * rb[c], src[c] + a * rb[c], rb[c]) for c in range(len(rb))
            for a in range(n)]
    columns = [(rt.column(t, c), rt.column(t, c) + N * rb[c]) for c in range(len(rb))]
    got = [g for g in got if any(a <= g[0] < b for a, b in columns)]  # without the priorities
    return [merged(got) == merged(want), len(rt.launches), words]


@pytest.mark.parametrize("how,elem_bytes,N,T,before,n", [
    ("managed", [1024, 32, 4], 500000, 200, 0, 500000),   # a whole 106 GB table, one run of slots
    ("managed", [1024, 32, 4], 500000, 200, 500000, 400000),
    ("ring", [2097169, 16], 65536, 1, 1000, 65536),       # wraps; priorities through a staging slot
    ("ring", [(1 << 28) + 8, 3], 512, 1, 200, 512),       # ... and in the launch's arguments
    ("ring", [1 << 30], 3, 100, 2, 2),                    # single rows of 100 GiB
    ("managed", [1 << 30], 3, 100, 2, 2),
    ("scattered", [2097169, 2097172, 2097168], 65536, 1, 0, 65536),
    ("scattered", [1 << 30], 20, 100, 0, 20),
    ("ring", [68, 24, 4, 4], 4096, 1000, 4000, 300),      # an ordinary call: one launch
])
def test_insertion(stub, how, elem_bytes, N, T, before, n):
    same, launches, words = stub_runtime.run(stub, __name__, "insertion", how, elem_bytes, N, T, before, n)
    assert same
    if how == "ring":
        assert words == (n if n <= 512 else 0)
    if elem_bytes[0] == 68:
        assert launches == 1


def gather(rt, elem_bytes, N, T, B, L, shift, fused):
    """Launches of one gather: their grids, and which bytes of each batch its pieces cover."""
    t = rt.table(elem_bytes, N, T)
    prio = np.ones(N, np.uint32)
    rt.gear.gear_insert(t, N, [rt.device(N * T * e) for e in elem_bytes], prio.ctypes.data)
    out = [rt.device(B * L * e + 16) + shift for e in elem_bytes]
    idx, start = rt.device(8 * B), rt.device(4 * B)
    del rt.launches[:]
    rt.reader = stub_runtime.read_collect
    try:
        if fused:
            rt.gear.gear_select_collect(t, rt.gear.GEAR_UNIFORM, B, L, 1, idx, start, 0, None, out)
        else:
            rt.gear.gear_collect(t, idx, start, B, L, None, out)
    except rt.gear.GearError as e:
        return [e.code, len(rt.launches)]
    covered = {}
    for name, grid, block, (unroll, task0, cols) in rt.launches:
        assert block == 256
        for k, c in enumerate(cols):
            # The column's pieces that this launch's workgroups take.
            first = max(0, -task0[k])
            stop = (task0[k + 1] if k + 1 < len(cols) else grid) - task0[k]
            stop = min(stop, grid - task0[k])
            piece = block * unroll * c["width"] if c["layout"] else c["wpp"] * c["W"]
            a, b = first * piece, min(stop * piece, B * c["W"])
            if a < b:
                covered.setdefault(c["out"], []).append((a, a, b - a))
    whole = all(merged(covered[o]) == [(0, 0, B * L * e)] for o, e in zip(out, elem_bytes))
    return [whole, len(rt.launches)]


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("elem_bytes,N,T,B,L,shift", [
    ([1024, 32, 4], 500000, 200, 1 << 20, 200, 0),   # 222 GB: beyond 128 GiB in 16-byte elements
    ([4112], 1 << 20, 4, 1 << 24, 1, 0),             # 69 GB of windows just above half a piece
    ([1028], 1 << 20, 200, 1 << 18, 200, 4),         # 54 GB written in 4-byte elements
    ([1025, 3], 1 << 16, 200, 1 << 16, 200, 1),      # 13 GB written in bytes
    ([1 << 30], 2, 150, 1, 150, 0),                  # one window of 150 GiB
    ([64, 4], 1000, 50, 256, 10, 0),                 # an ordinary call: one launch
])
def test_gather(stub, elem_bytes, N, T, B, L, shift, fused):
    whole, launches = stub_runtime.run(stub, __name__, "gather", elem_bytes, N, T, B, L, shift, fused)
    assert whole is True
    assert (launches == 1) == (B == 256)


def test_a_refused_gather_launches_nothing(stub):
    """The second group of 16 columns has 2^31 pieces or more: 20 TB of windows."""
    assert stub_runtime.run(stub, __name__, "gather", [4] * 16 + [1 << 20], 1 << 20, 4, 1 << 24, 1, 0, False) == [-1, 0]
