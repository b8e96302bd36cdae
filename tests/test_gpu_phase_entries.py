"""Phase ops whose factors of the thread come in every number around the step in
which the kernels read them: one-qubit diagonals, CZ pairs and Z strings on qubits
off the registers, and strings across them; states and gradients against the oracle.

Bars as for other fused plans: 1e-12 (c128) / 1e-5 (c64); gradients 1e-11 / 2e-5 x
sum|alpha|.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_13524_amd import Batch, Circuit, Observable, Plan, State, adjoint_gradient, apply_fused
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu

AMP_TOL = {"c128": 1e-12, "c64": 1e-5}
RED_TOL = {"c128": 1e-11, "c64": 2e-5}


def circuit(n, k, seed):
    rng = np.random.default_rng((n, k, seed))
    gates, slot = [{"op": "h", "q": [q]} for q in range(n)], 0
    pairs = [(a, b) for a in range(n) for b in range(a + 1, n)]
    for layer in range(2):
        for q in rng.permutation(n)[:k]:
            gates.append({"op": "rz", "q": [int(q)], "slot": slot})
            slot += 1
        for i in rng.permutation(len(pairs))[:k]:
            gates.append({"op": "cz", "q": list(pairs[i])})
        for i in rng.permutation(len(pairs))[:k]:
            gates.append({"op": "pauli_rot", "q": list(pairs[i]), "paulis": [3, 3], "slot": slot})
            slot += 1
        gates.append({"op": "pauli_rot", "q": [int(x) for x in rng.permutation(n)[:4]], "paulis": [3] * 4, "angle": 0.3})
        for q in range(n):  # a rotation on every qubit: the phases are due
            gates.append({"op": ("rx", "ry")[(q + layer) % 2], "q": [q], "slot": slot})
            slot += 1
    return gates, slot


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9])
def test_every_number_of_entries(dt, k):
    for n in (9, 12, 14):
        gates, npar = circuit(n, k, 1)
        theta = np.random.default_rng(k).uniform(-7.0, 7.0, npar)
        c = Circuit.from_records(n, gates)
        s, plan = State(n, dt), Plan(c, dt)
        apply_fused(s, plan, theta)
        assert np.max(np.abs(s.store() - O.run_circuit(n, gates, theta))) <= AMP_TOL[dt], n
        obs = W.random_pauli_observable(n, 8, (1, 3), seed_key=(n, k)) + [(0.4, [])]
        scale = sum(abs(a) for a, _ in obs)
        slots = [0, npar // 2, npar - 1]
        ref = O.param_shift_grad(n, gates, theta, obs, slots=slots)
        psi, lam, b = State(n, dt), State(n, dt), Batch()
        b.add(c, Observable(n, obs), theta)
        be, bg = b.run(dt)
        for e, g in [adjoint_gradient(c, theta, Observable(n, obs), psi, lam, plan), (be[0], bg[0])]:
            assert abs(e - O.energy(n, gates, theta, obs)) <= RED_TOL[dt] * scale
            assert np.max(np.abs(g[slots] - ref)) <= RED_TOL[dt] * scale
