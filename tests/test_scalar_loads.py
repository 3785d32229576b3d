"""Every scalar load of the library has an aligned offset.

A scalar load drops the two lowest bits of each part of its address, the base
and the offset, not of their sum.  The compiler once read a pointer out of a
kernel argument struct with a base of 14 and an offset of 0x32, an aligned sum
of two unaligned parts (one induction variable served as a shift count and as a
byte offset), and the kernel added into a wild address.  An unaligned offset is
the visible half of such a pair (CPU only: hipcc cross-compiles)."""
import os
import re
import subprocess

import pytest

from paper_2310_05205_amd import build

LOAD = re.compile(r"^\s*(s_(?:buffer_)?load_dword\S*\s.*)$", re.M)


@pytest.mark.parametrize("source", build.SOURCES)
def test_scalar_load_offsets_are_aligned(source, tmp_path):
    hipcc = os.environ.get("HIPCC", "hipcc")
    out = tmp_path / "listing.s"
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S", "-o", str(out),
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + build.INCLUDE, "-I" + build.CSRC, os.path.join(build.CSRC, source)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    loads = LOAD.findall(out.read_text())
    if source != "table.hip":  # host-only code, no kernels
        assert loads
    bad = []
    for line in loads:
        for x in re.findall(r"(?:,\s*|offset:)(0x[0-9a-f]+|\d+)\s*(?:;.*)?$", line):
            if int(x, 0) % 4:
                bad.append(line)
    assert bad == []
