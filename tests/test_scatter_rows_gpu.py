"""Row writes in scattered slot order, against rows written by numpy.

Rows around the scatter kernels' 1 KiB piece in elements of 1, 4 and 16 bytes:
one piece or several, last pieces of one element, of all but one and whole, and
rows of half a piece, where the kernel for small rows ends.  Only some slots are
written, so bytes that a piece puts behind its row stay visible."""
import numpy as np
import pytest
import torch

from paper_2310_05205_amd import gear
from tests.helpers import cuda, host, say

pytestmark = pytest.mark.gpu

# Row bytes; 4-byte elements unless 16 divides them, 1-byte ones when 4 does not.
ROWS = [508, 512, 516, 1020, 1024, 1028, 2044, 2052, 2136, 3076, 511, 513, 534, 1023, 1025, 2049, 528, 1040, 2064]


@pytest.mark.parametrize("shift", [0, 4, 1])
@pytest.mark.parametrize("row", ROWS)
def test_scattered_rows(row, shift):
    N, n = 97, 60
    rng = np.random.default_rng(row + shift)
    t = gear.Table([row], N, 1)
    try:
        model = rng.integers(0, 256, (N, row), dtype=np.uint8)
        t.insert([model], np.ones(N, np.uint32))
        for step in range(2):
            say("row %d shift %d step %d" % (row, shift, step))
            idx = np.concatenate([[N - 1], rng.permutation(N - 1)[:n - 1]])[rng.permutation(n)].astype(np.int64)
            data = rng.integers(0, 256, (n, row), dtype=np.uint8)
            buf = torch.zeros(n * row + 4096, dtype=torch.uint8, device=cuda())
            buf[shift:shift + n * row] = torch.from_numpy(data.reshape(-1)).to(cuda())
            t.write_rows(idx, [buf[shift:shift + n * row].view(n, row)])
            model[idx] = data
            np.testing.assert_array_equal(host(t.column_view(0)), model)
    finally:
        t.close()
