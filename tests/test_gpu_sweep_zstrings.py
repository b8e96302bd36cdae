"""Adjoint gradients with a forward plan of circuits with parametric Z strings, over
the sweep's shapes: LDS passes (3 to 8 qubits), one register tile, several.

Bars as for the other gradients: 1e-11 (c128) / 2e-5 (c64) x sum|alpha|.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_13524_amd import Circuit, Observable, Plan, State, adjoint_gradient
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu

RED_TOL = {"c128": 1e-11, "c64": 2e-5}


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n", [3, 4, 5, 8, 9, 11, 12, 13])
def test_plan_backed_gradient_of_a_qaoa_circuit(dt, n):
    rng = np.random.default_rng(n)
    gates, slot = [{"op": "h", "q": [q]} for q in range(n)], 0
    for _ in range(2):
        for q in range(n):
            w = int(rng.integers(2, min(n, 5) + 1))
            gates.append({"op": "pauli_rot", "q": [int(x) for x in rng.permutation(n)[:w]], "paulis": [3] * w, "slot": slot})
            slot += 1
        for q in range(n):
            gates.append({"op": ("rx", "ry")[q % 2], "q": [q], "slot": slot})
            slot += 1
    obs = W.random_pauli_observable(n, 12, (1, min(n, 4)), seed_key=(n, 4)) + [(0.4, [])]
    scale = sum(abs(c) for c, _ in obs)
    circ, o = Circuit.from_records(n, gates), Observable(n, obs)
    plan = Plan(circ, dt)
    for k in range(2):
        theta = np.random.default_rng((n, k)).uniform(-7.0, 7.0, slot)
        psi, lam = State(n, dt), State(n, dt)
        e, g = adjoint_gradient(circ, theta, o, psi, lam, plan)
        assert abs(e - O.energy(n, gates, theta, obs)) <= RED_TOL[dt] * scale
        ref = O.param_shift_grad(n, gates, theta, obs, slots=list(range(slot)))
        assert np.max(np.abs(g - ref)) <= RED_TOL[dt] * scale
