"""Every scalar condition of the library has a setter that can have meant it.

A scalar select, branch or add with carry reads SCC, which scalar instructions
set and vector compares do not.  The compiler once turned a uniform 64-bit
comparison into a vector compare, branched on that, and behind the branch selected
by an SCC that the last scalar addition had left: a row's short last piece was
copied whole.  For every reader of SCC the last setter on each path to it must be a
comparison, a logical operation (whose SCC says that the result is not zero) or
the addition or subtraction whose carry is meant (CPU only: hipcc
cross-compiles)."""
import os
import re
import subprocess

import pytest

from paper_2310_05205_amd import build

READS = re.compile(r"s_(cselect|cmov|cbranch_scc|addc_u32|subb_u32)")
SETS = re.compile(r"s_(cmpk?_|bitcmp|add_|sub_|addc_|subb_|addk_|and_|or_|xor_|andn[12]_|orn[12]_|nand_|nor_|xnor_|not_|"
                  r"lshl|lshr_|ashr_|bfe_|min_|max_|abs|bcnt|wqm|quadmask|\w+_saveexec)")
CARRY = re.compile(r"s_(add_u32|sub_u32|addc_u32|subb_u32|cmp)")
MEANT = re.compile(r"s_(cmp|bitcmp|and_|or_|xor_|andn|orn|nand_|nor_|xnor_|not_|\w+_saveexec|add_u32|sub_u32|addc_u32|"
                   r"subb_u32|lshl_b|lshr_b)")


def _functions(listing):
    """{name: [block]}, a block as (labels, instructions, falls through)."""
    out, name, blocks = {}, None, None
    for line in listing.splitlines():
        text = line.split(";")[0].strip()
        start = re.match(r"(_Z\w+):", line)
        if start:
            name = start.group(1)
            blocks = out[name] = [([], [])]
        elif name is None:
            continue
        elif text.startswith(".amdhsa_kernel"):
            name = None
        elif re.match(r"\.LBB\w+:", line):
            blocks.append(([line.split(":")[0]], []))
        elif line.startswith("; %bb."):
            blocks.append(([], []))
        elif text and not text.startswith("."):
            blocks[-1][1].append(text)
    return out


def _setters(blocks, k, seen):
    """The last setters of SCC on the paths that end before block k."""
    found = set()
    labels = blocks[k][0]
    for j, (_, code) in enumerate(blocks):
        jumps = [c for c in code if c.startswith("s_cbranch") or c.startswith("s_branch")]
        falls = j + 1 == k and not (code and re.match(r"s_(branch|endpgm)", code[-1]))
        if not falls and not any(c.split()[-1] in labels for c in jumps):
            continue
        sets = [c for c in code if SETS.match(c)]
        if sets:
            found.add(sets[-1])
        elif j not in seen:
            found |= _setters(blocks, j, seen | {j})
    return found


def unset_conditions(listing):
    bad = []
    for name, blocks in _functions(listing).items():
        for k, (_, code) in enumerate(blocks):
            last = None
            for c in code:
                if READS.match(c):
                    setters = {last} if last else _setters(blocks, k, {k})
                    fits = CARRY if re.match(r"s_(addc|subb)", c) else MEANT
                    if not setters or not all(fits.match(s) for s in setters):
                        bad.append((name, c, sorted(setters)))
                if SETS.match(c):
                    last = c
    return bad


@pytest.mark.parametrize("source", [s for s in build.SOURCES if s != "table.hip"])  # table.hip has no kernels
def test_scalar_conditions_are_set(source, tmp_path):
    hipcc = os.environ.get("HIPCC", "hipcc")
    out = tmp_path / "listing.s"
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S", "-o", str(out),
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + build.INCLUDE, "-I" + build.CSRC, os.path.join(build.CSRC, source)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = out.read_text()
    assert READS.search(text)
    assert unset_conditions(text) == []
