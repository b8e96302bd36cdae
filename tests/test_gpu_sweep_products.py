"""Precision of the products in the reverse sweep: from the same complex64 states, the
gradient of a rotation below 20 qubits is their FP64 sum, not one of FP32 products.

The last gate of the circuit is the parametric one, on qubit 0, so its term is taken
from psi and lambda - E psi as they come: the states of the same plan and of
apply_observable, shifted in complex64 with one rounding (E in complex64). The bar
is FP64 rounding with room for a shift rounded twice here: 1e-12 x sum|alpha|;
products in FP32 are off by 1e-9 and more.
"""
import numpy as np
import pytest

from paper_2011_13524_amd import Circuit, Observable, Plan, State, adjoint_gradient, apply_fused, apply_observable
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["rx", "ry"])
@pytest.mark.parametrize("n", [9, 10, 11, 12, 13, 15])
def test_last_rotation(n, op):
    rng = np.random.default_rng(n)
    gates = []
    for layer in range(3):
        gates += [{"op": ("rx", "ry", "rz")[(q + layer) % 3], "q": [q], "angle": float(rng.uniform(-3, 3))} for q in range(n)]
        gates += [{"op": "cnot", "q": [q, (q + 1) % n]} for q in range(n)]
    gates.append({"op": op, "q": [0], "slot": 0})
    theta = np.array([0.7])
    obs = W.random_pauli_observable(n, 20, (1, 4), seed_key=(n, 8))
    scale = sum(abs(a) for a, _ in obs)
    c, o = Circuit.from_records(n, gates), Observable(n, obs)
    plan = Plan(c, "c64")
    s, t, psi, lam = (State(n, "c64") for _ in range(4))
    apply_fused(s, plan, theta)
    apply_observable(s, o, t)
    a, b = (np.asarray(x.store()).astype(np.complex128) for x in (s, t))
    e, g = adjoint_gradient(c, theta, o, psi, lam, plan)
    e32 = float(np.float32(e))
    b = (b - e32 * a).astype(np.complex64).astype(np.complex128)
    p = a.reshape(-1, 2)[:, ::-1] * (np.array([1.0, 1.0]) if op == "rx" else np.array([-1j, 1j]))
    ref = -np.vdot(b, p.reshape(-1)).imag / np.sum(np.abs(a) ** 2)
    assert abs(g[0] - ref) <= 1e-12 * scale
