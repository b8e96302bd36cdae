"""Expectations whose passes run in one launch with their groups split over
workgroups: few tiles and many strings, one tile and several, records of every
kind, ragged ranges of tiles; against the oracle, and twice the same bits.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_13524_amd import Observable, State, apply_observable, expectation
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu

# per unit of sum |alpha|: FP64 sums of products (c128); a product and a sum of
# at most 8 in FP32, 9 x 2^-24 = 5.4e-7 (c64), with the amplitudes' own rounding
# taken out by giving the oracle the rounded state
TOL = {"c128": 1e-13, "c64": 6e-7}


@pytest.mark.parametrize("grid", [None, "3"])
@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,terms", [(2, 3), (7, 60), (11, 1), (12, 300), (13, 300), (13, 700), (15, 40), (16, 300)])
def test_split_passes_vs_oracle(dt, n, terms, grid, monkeypatch):
    if grid:
        monkeypatch.setenv("QSV_EXPECT_GRID", grid)
    rng = np.random.default_rng((n, terms))
    v = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    v /= np.linalg.norm(v)
    if dt == "c64":
        v = v.astype(np.complex64).astype(np.complex128)
    obs = W.random_pauli_observable(n, terms, (1, min(n, 5)), seed_key=(n, terms)) + [(0.3, [])]
    obs += [(0.1 * (k + 1), [(q, 3) for q in range(k + 1)]) for k in range(min(n, 12))]  # one mask, many terms
    s = State(n, dt)
    s.load(v)
    got = expectation(s, Observable(n, obs))
    assert abs(got - O.expectation(v, obs)) <= TOL[dt] * sum(abs(c) for c, _ in obs)
    assert expectation(s, Observable(n, obs)) == got


@pytest.mark.parametrize("grid", [None, "3"])
@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,terms", [(11, 60), (12, 300), (13, 300), (13, 700), (15, 200)])
def test_lambda_records_vs_oracle(dt, n, terms, grid, monkeypatch):
    # lambda = O psi, all kinds of strings; every amplitude sums up to `terms`
    # products in the state's precision
    if grid:
        monkeypatch.setenv("QSV_EXPECT_GRID", grid)
    rng = np.random.default_rng((n, terms, 2))
    v = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    v /= np.linalg.norm(v)
    if dt == "c64":
        v = v.astype(np.complex64).astype(np.complex128)
    obs = W.random_pauli_observable(n, terms, (1, 6), seed_key=(n, terms, 2)) + [(0.3, [])]
    obs += [(0.1 * (k + 1), [(q, 3) for q in range(k + 1)]) for k in range(min(n, 12))]
    ref = O.apply_observable(v, obs)
    s, out = State(n, dt), State(n, dt)
    s.load(v)
    apply_observable(s, Observable(n, obs), out)
    scale = sum(abs(c) for c, _ in obs) * np.max(np.abs(v))
    # each product and sum rounds by 2^-24 (2^-53) of at most the running sum
    tol = (terms + 20) * (2.0**-23 if dt == "c64" else 2.0**-52)
    assert np.max(np.abs(out.store() - ref)) <= tol * scale
