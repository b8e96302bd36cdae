"""Rounding of one-qubit unitaries in fused plans: ten layers of Haar gates and CZ in
complex128. Each layer multiplies every amplitude by rounded sums of two products (about
2.5 units of 2^-53 rms with the matrix entries as they come): rms 1.4e-15 over ten
layers, bar twice that. The same error on every amplitude, as from rounded factors of
a matrix, adds up to several times as much.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_13524_amd import Circuit, Plan, State, apply_fused
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [9, 11, 12, 14])
def test_haar_layers(n):
    for seed in range(3):
        rng = np.random.default_rng((n, seed))
        gates = []
        for _ in range(10):
            gates += [{"op": "dense", "q": [q], "mat": W.haar_unitary(rng, 2)} for q in range(n)]
            p = [int(x) for x in rng.permutation(n)]
            gates += [{"op": "cz", "q": [p[2 * j], p[2 * j + 1]]} for j in range(n // 2)]
        s = State(n, "c128")
        apply_fused(s, Plan(Circuit.from_records(n, gates), "c128"))
        ref = O.run_circuit(n, gates)
        assert np.linalg.norm(s.store() - ref) <= 2.8e-15 + 1.4e-15  # (the oracle's own rounding)
