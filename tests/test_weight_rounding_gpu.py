"""Importance-sampling weights next to the middle of two fp32 numbers.

At beta 1 the weight is the fp64 quotient of two priorities, rounded to fp32.  Here
that quotient lies 2 to 4 units in its last place from half way between two fp32
numbers, so a power that is wrong by more than its own rounding gives the other
one.  pow is within one unit; exp(beta * log(m / p)) loses the low bits of the
logarithm, about 9 here, and is off by up to 8."""
import random

import numpy as np
import pytest
import torch

from paper_2310_05205_amd import gear
from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu

SHIFT = 38  # the middles are k / 2^38, k odd with 25 bits: weights near 2^-13


def _pairs(count):
    """(m, p) with m / p next to k / 2^SHIFT: m * 2^SHIFT - k * p is a small c."""
    rng = random.Random(5)
    out = []
    while len(out) < count:
        k = rng.randrange(1 << 24, 1 << 25) | 1
        c = rng.choice((-1, 1)) * rng.randrange(1, 80)
        p = -c * pow(k, -1, 1 << SHIFT) % (1 << SHIFT)
        m = (k * p + c) >> SHIFT
        if not 1 <= m < p < 1 << 32:
            continue
        x, middle = np.float64(m) / np.float64(p), np.ldexp(float(k), -SHIFT)
        if 2 <= abs(x - middle) / np.spacing(middle) <= 4:
            out.append((m, p, np.float32(x)))
    return out


def test_shared_weights():
    t = gear.Table([], 16, 1)
    try:
        pairs = _pairs(200)
        got = [host(t.is_weights(torch.from_numpy(np.array([m, p], np.uint32).view(np.int32)).to(cuda()), 1.0))[1]
               for m, p, _ in pairs]
        np.testing.assert_array_equal(np.array(got), np.array([w for _, _, w in pairs]))
    finally:
        t.close()


@pytest.mark.parametrize("N", [64, 40000])  # one launch, and search and weight kernels
def test_selected_weights(N):
    for m, p, want in _pairs(30):
        t = gear.Table([], N, 1)
        try:
            t.set_options(gear.GEAR_OPT_IS_GLOBAL_MIN)
            prio = np.zeros(N, np.uint32)
            prio[[3, N - 1]] = m, p
            t.insert([], prio)
            idx, _, w = t.select(gear.GEAR_PRIORITIZED, 8, 1, 1, 1.0, weights=True)
            np.testing.assert_array_equal(host(idx), N - 1)
            np.testing.assert_array_equal(host(w), want)
        finally:
            t.close()
