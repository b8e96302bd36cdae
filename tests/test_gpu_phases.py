"""Register-resident passes: phases (diagonal factors merged over register bits,
thread bits and non-local qubits), rotations by shears and exchanges, against
the CPU oracle.

Bars as for other fused plans: amplitudes max-abs 1e-12 (c128) / 1e-5 (c64);
gradients 1e-11 / 2e-5 x sum|alpha| (rounding grows with the gate count only).
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_13524_amd import Circuit, Observable, Plan, State, adjoint_gradient, apply_fused
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu

AMP_TOL = {"c128": 1e-12, "c64": 1e-5}
RED_TOL = {"c128": 1e-11, "c64": 2e-5}
# (dtype, thread bits, tile qubits): every register shape
SHAPES = [("c128", "8", 0), ("c128", "7", 11), ("c64", "8", 0), ("c64", "9", 13), ("c64", "8", 13), ("c64", "7", 11)]


def phase_circuit(n, count, seed, parametric=False):
    """Diagonals of every kind between rotations, exchanges and products."""
    rng = np.random.default_rng(seed)
    g, slot = [], 0
    for _ in range(count):
        r = int(rng.integers(0, 12))
        q = [int(x) for x in rng.permutation(n)[:5]]
        ang = float(rng.uniform(-6.3, 6.3))
        if r <= 2:  # Z strings of weight 1..5
            w = int(rng.integers(1, 6))
            rec = {"op": "pauli_rot", "q": q[:w], "paulis": [3] * w, "angle": ang}
        elif r == 3:
            rec = {"op": "rz", "q": q[:1], "angle": ang}
        elif r == 4:
            rec = {"op": "cz", "q": q[:2]}
        elif r <= 7:
            rec = {"op": "rx" if r < 7 else "ry", "q": q[:1], "angle": ang}
        elif r == 8:
            rec = {"op": "cnot", "q": q[:2]}
        elif r == 9:  # X with a control that is 0, and with two controls
            c = int(rng.integers(1, 3))
            rec = {"op": "dense", "q": q[:1], "mat": np.array([[0, 1], [1, 0]]), "controls": q[1:1 + c],
                   "ctrl_vals": [int(v) for v in rng.integers(0, 2, c)]}
        elif r == 10:
            rec = {"op": "h", "q": q[:1]}
        else:
            rec = {"op": "dense", "q": q[:1], "mat": W.haar_unitary(rng, 2)}
        if parametric and "angle" in rec:
            del rec["angle"]
            rec["slot"] = slot
            slot += 1
        g.append(rec)
    return g, slot


@pytest.mark.parametrize("dt,tb,tile", SHAPES)
@pytest.mark.parametrize("heavy", [False, True])
def test_phases_in_every_register_shape(dt, tb, tile, heavy, monkeypatch):
    monkeypatch.setenv("QSV_TILE_THREAD_BITS", tb)
    for n, seed in ((13, 1), (15, 2)):
        gates, _ = phase_circuit(n, 260, seed)
        # a last layer of diagonals only: flushed at the end, off the registers too
        for a in range(n):
            gates.append({"op": "rz", "q": [a], "angle": 0.1 + 0.2 * a})
            gates.append({"op": "cz", "q": [a, (a + 5) % n]})
            gates.append({"op": "pauli_rot", "q": [a, (a + 1) % n], "paulis": [3, 3], "angle": 0.3 * a - 1.0})
        p = Plan(Circuit.from_records(n, gates), dt, tile_qubits=tile, heavy=heavy)
        assert p.info()["segments"] > 0
        s = State(n, dt)
        apply_fused(s, p)
        assert np.max(np.abs(s.store() - O.run_circuit(n, gates))) <= AMP_TOL[dt], (n, p.info())


@pytest.mark.parametrize("dt", ["c128", "c64"])
def test_matrices_off_unitary_keep_the_general_product(dt):
    # a one-qubit matrix that is not unitary (by a little, and by a lot) and a
    # diagonal that is not of modulus one
    n = 13
    rng = np.random.default_rng(5)
    gates = [{"op": "h", "q": [q]} for q in range(n)]
    for q in range(n):
        u = W.haar_unitary(rng, 2)
        gates.append({"op": "dense", "q": [q], "mat": u * (1.0 + 1e-6 * (q == 3)) + (0.05 if q % 2 else 1e-7) * np.eye(2)})
        gates.append({"op": "dense", "q": [q], "mat": np.diag([1.02, 0.9 + 0.1j])})
        gates.append({"op": "cnot", "q": [q, (q + 4) % n]})
    s = State(n, dt)
    apply_fused(s, Plan(Circuit.from_records(n, gates), dt))
    ref = O.run_circuit(n, gates)
    assert np.max(np.abs(s.store() - ref)) <= AMP_TOL[dt] * max(1.0, float(np.max(np.abs(ref))))


@pytest.mark.parametrize("dt", ["c128", "c64"])
def test_parametric_phases_follow_theta_and_differentiate(dt, monkeypatch):
    monkeypatch.setenv("QSV_ADJOINT_TILED_MIN", "1")
    n = 13
    gates, npar = phase_circuit(n, 90, 7, parametric=True)
    c = Circuit.from_records(n, gates)
    plan = Plan(c, dt)
    obs = W.random_pauli_observable(n, 12, (1, 3), seed_key=(8, n))
    scale = sum(abs(a) for a, _ in obs)
    s = State(n, dt)
    for seed in (1, 2):  # the plan's values are formed anew for each theta
        theta = np.random.default_rng(seed).uniform(-7.0, 7.0, npar)
        s.set_basis(0)
        apply_fused(s, plan, theta)
        assert np.max(np.abs(s.store() - O.run_circuit(n, gates, theta))) <= AMP_TOL[dt]
    psi, lam = State(n, dt), State(n, dt)
    e, g = adjoint_gradient(c, theta, Observable(n, obs), psi, lam, plan)
    ref = O.param_shift_grad(n, gates, theta, obs, slots=list(range(npar)))
    assert abs(e - O.energy(n, gates, theta, obs)) <= RED_TOL[dt] * scale
    assert np.max(np.abs(g - ref)) <= RED_TOL[dt] * scale
    # psi is uncomputed to |0...0>, its sign included
    assert abs(psi.store()[0] - 1.0) <= 10 * AMP_TOL[dt]


@pytest.mark.parametrize("dt,n", [("c64", 5), ("c64", 8), ("c64", 9), ("c64", 10), ("c64", 11), ("c64", 12), ("c64", 13),
                                  ("c128", 6), ("c128", 8), ("c128", 9), ("c128", 10), ("c128", 11), ("c128", 12)])
def test_gradients_around_the_smallest_full_tile(dt, n):
    # every register shape, one tile and two, and the LDS sweep below; then with a
    # gate of more local controls than the passes take (the per-gate sweep does)
    rng = np.random.default_rng(n)
    g, npar = phase_circuit(n, 50, 5 + n, parametric=True)
    ctrl = {"op": "dense", "q": [0], "mat": W.haar_unitary(rng, 2), "controls": list(range(1, n)),
            "ctrl_vals": [int(v) for v in rng.integers(0, 2, n - 1)]}
    obs = W.random_pauli_observable(n, 12, (1, 4), seed_key=(n, 3)) + [(0.4, [])]
    theta = rng.uniform(-6.3, 6.3, npar)
    scale = sum(abs(c) for c, _ in obs)
    for gates in (g, g[:25] + [ctrl] + g[25:]):
        psi, lam = State(n, dt), State(n, dt)
        e, gr = adjoint_gradient(Circuit.from_records(n, gates), theta, Observable(n, obs), psi, lam)
        assert abs(e - O.energy(n, gates, theta, obs)) <= RED_TOL[dt] * scale
        slots = sorted({0, 1, npar // 2, npar - 1})
        ref = O.param_shift_grad(n, gates, theta, obs, slots=slots)
        assert np.max(np.abs(gr[slots] - ref)) <= RED_TOL[dt] * scale


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("max_k", [2, 3, 5])
def test_states_of_one_tile(dt, n, max_k):
    # three register bits below 12 qubits; blocks of up to max_k qubits too
    g, _ = phase_circuit(n, 90, 40 + n)
    rng = np.random.default_rng(n)
    for k in (2, 3):
        g.insert(30 * k, {"op": "dense", "q": [int(x) for x in rng.permutation(n)[:k]], "mat": W.haar_unitary(rng, 1 << k)})
    v = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    v /= np.linalg.norm(v)
    s = State(n, dt)
    s.load(v)
    ref = v.astype(np.complex64).astype(np.complex128) if dt == "c64" else v.copy()
    apply_fused(s, Plan(Circuit.from_records(n, g), dt, max_k=max_k))
    for rec in g:
        O.apply_gate(ref, rec, None)
    assert np.max(np.abs(s.store() - ref)) <= AMP_TOL[dt]


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("strings", ["z", "xy"])
def test_sweep_tables_kept_with_a_plan(dt, strings):
    # one plan, several parameter vectors and states: with the tables kept from
    # the first gradient (Z strings only) and without (strings with X and Y)
    n = 13
    g, npar = phase_circuit(n, 60, 77, parametric=True)
    g = g + [{"op": "pauli_rot", "q": [1, 5, 12], "paulis": [3, 3, 3] if strings == "z" else [1, 2, 3], "slot": npar}]
    npar += 1
    obs = W.random_pauli_observable(n, 12, (1, 4), seed_key=(n, 9)) + [(0.4, [])]
    scale = sum(abs(c) for c, _ in obs)
    circ, o = Circuit.from_records(n, g), Observable(n, obs)
    plan = Plan(circ, dt)
    slots = [0, npar // 3, npar - 2, npar - 1]
    for k in range(3):
        theta = np.random.default_rng(k).uniform(-7.0, 7.0, npar)
        psi, lam = State(n, dt), State(n, dt)
        e, gr = adjoint_gradient(circ, theta, o, psi, lam, plan)
        assert abs(e - O.energy(n, g, theta, obs)) <= RED_TOL[dt] * scale
        ref = O.param_shift_grad(n, g, theta, obs, slots=slots)
        assert np.max(np.abs(gr[slots] - ref)) <= RED_TOL[dt] * scale


@pytest.mark.parametrize("tb", ["7", "8", "9"])
@pytest.mark.parametrize("n", [8, 9, 10, 11, 12])
def test_one_tile_under_every_thread_bits_setting(n, tb, monkeypatch):
    # shapes that are not compiled (9 thread bits at 12 qubits, 7 at 9) fall back
    monkeypatch.setenv("QSV_TILE_THREAD_BITS", tb)
    g, _ = phase_circuit(n, 40, 60 + n)
    for dt in ("c64", "c128"):
        s = State(n, dt)
        apply_fused(s, Plan(Circuit.from_records(n, g), dt))
        assert np.max(np.abs(s.store() - O.run_circuit(n, g))) <= AMP_TOL[dt]
