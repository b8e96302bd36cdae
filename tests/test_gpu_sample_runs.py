"""Sampling through a table of every 16th value: states of less than one run, of
part of a chunk, of one chunk and of several, with runs of probability zero, the
ends of [0, 1), and uniforms that fall exactly on a value of the scan.
"""
import numpy as np
import pytest

from paper_2011_13524_amd import State

pytestmark = pytest.mark.gpu


def scan(p):
    """The cumulative sums as the table forms them: runs of 16 in order, offsets
    of a chunk of 4096 in order (exact here: multiples of 2^-k)."""
    return np.cumsum(p)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 9, 12, 13, 15])
def test_draws_equal_the_inverse_of_the_scan(dt, n):
    rng = np.random.default_rng(n)
    # amplitudes 0, 1/2, 1: every sum is exact, so every draw is determined
    v = rng.integers(0, 3, 1 << n) / 2.0
    v[rng.random(1 << n) < 0.4] = 0.0
    if n >= 9:
        v[64:160] = 0.0  # whole runs of probability zero
    v[-1 if n % 2 else 0] = 1.0
    s = State(n, dt)
    s.load(v * (1j if n % 3 == 0 else 1.0))
    c = scan(v * v)
    total = c[-1]
    k = rng.integers(0, 1 << 20, 3000) / float(1 << 20)
    at = c[rng.integers(0, 1 << n, 200)] / total  # near or on a value of the scan
    u = np.concatenate([k, at[at < 1.0], [0.0, 1.0 - 2.0**-53]])
    want = np.searchsorted(c, u * total, side="right")
    got = s.sample(u)
    assert np.array_equal(got, np.minimum(want, np.nonzero(v)[0][-1]))
