"""Kernels read page-locked host memory at its device address.

Memory that the caller page-locks after allocating it may have another address on
the device than on the host; a kernel that reads the host's would fault.  The
calls run on the CPU over a runtime whose locked memory lies elsewhere on the
device, and every pointer that a launch receives must be the device's."""
import ctypes

import numpy as np
import pytest

from tests import stub_runtime


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return stub_runtime.build(tmp_path_factory.mktemp("stub"))


def addresses(rt, how, n):
    """Offsets into the locked rows and priorities that the launches read at, or None for a host address."""
    gear, E, N = rt.gear, 2052, 3000
    t = rt.table([E], N, 1)
    rows, prio = np.zeros(n * E, np.uint8), np.ones(n, np.uint32)
    for a in (rows, prio):
        rt.stub.stub_lock(a.ctypes.data, a.nbytes)
    rows_on_device = rt.device(n * E)
    offset = rt.stub.stub_locked_offset()
    seen = []

    def reader(name, args):
        if "copy_segments" in name:
            task0, seg, _ = stub_runtime.read_segments(name, args)
            seen.extend(s for k, (s, _, _) in enumerate(seg) if task0[k] != 0xFFFFFFFF)
        elif "scatter_rows" in name or "commit_kernel" in name:
            seen.append(ctypes.cast(args[1], ctypes.POINTER(ctypes.c_uint64)).contents.value)

    rt.reader = reader
    if how == "ring":
        gear.gear_insert(t, n, [rows_on_device], prio.ctypes.data)
    else:
        gear.gear_table_use_allocator(t, gear.GEAR_FIFO, N)
        idx = gear.gear_allocate(t, n)
        gear.gear_write_rows(t, idx[::-1] if how == "scattered" else idx, [rows.ctypes.data])
        gear.gear_commit(t, idx, prio.ctypes.data)
    spaces = {"rows": rows, "prio": prio}
    out = []
    for s in seen:
        if rows_on_device <= s < rows_on_device + n * E:
            continue
        out.append([[k, s - offset - a.ctypes.data] for k, a in spaces.items()
                    if 0 <= s - offset - a.ctypes.data < a.nbytes])
    return out


@pytest.mark.parametrize("how,n,want", [
    ("ring", 100, [[["prio", 0]]]),
    ("ring", 3100, [[["prio", 400]], [["prio", 12000]]]),   # the last 3000 rows, in two parts of the ring
    ("slots", 100, [[["rows", 0]], [["prio", 0]]]),
    ("scattered", 100, [[["rows", 0]], [["prio", 0]]]),
])
def test_locked_sources(stub, how, n, want):
    assert stub_runtime.run(stub, __name__, "addresses", how, n) == want
