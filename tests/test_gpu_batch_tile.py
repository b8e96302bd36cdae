"""Batch items that run as tile passes over all items at once: the smallest size
that takes the path and the ones around it, with Z strings, fixed and shared
parameters, general one-qubit gates, observables with X, Y and Z factors, and
items of the other path between them; energies and gradients against the oracle.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_13524_amd import Batch, Circuit, Observable
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu

# relative to the observable's norm: ~120 operations, each rounding once or
# twice (2^-53, 2^-24), errors adding like their root; the double bound is the
# batch tests' own
TOL = {"c128": 1e-10, "c64": 2e-5}


def item(n, k):
    rng = np.random.default_rng((n, k))
    gates, slot = [], 0
    for q in range(n):
        gates.append({"op": "h", "q": [q]} if q % 3 else {"op": "rx", "q": [q], "angle": 0.2 + 0.1 * q})
    for layer in range(2):
        for q in range(n):
            gates.append({"op": ("rx", "ry", "rz")[int(rng.integers(3))], "q": [q], "slot": slot})
            slot += 1
        for q in range(0, n - 1, 2):
            a, b = (q, q + 1) if rng.random() < 0.5 else (q + 1, q)
            gates.append({"op": "cnot" if (q // 2 + layer) % 2 else "cz", "q": [a, b]})
        gates.append({"op": "pauli_rot", "q": [0, n // 2, n - 1], "paulis": [3, 3, 3], "slot": slot})
        slot += 1
        gates.append({"op": "ry", "q": [n - 1], "slot": 0})  # a parameter used twice
        gates.append({"op": "rz", "q": [n // 2], "angle": -0.7})
    theta = rng.uniform(-7.0, 7.0, slot)  # beyond one turn
    obs = W.random_pauli_observable(n, 12, (1, 4), seed_key=(n, k)) + [(0.4, [])]
    return n, gates, theta, obs


def shift_rule(n, gates, theta, obs, slots):
    """The oracle's shift rule takes a slot per gate: later uses of a slot get
    their own, and the gradient is the sum over the uses."""
    seen, uses, own, th = set(), {}, [], list(theta)
    for g in gates:
        if "slot" in g:
            s = t = g["slot"]
            if s in seen:
                t = len(th)
                th.append(theta[s])
            seen.add(s)
            uses.setdefault(s, []).append(t)
            g = dict(g, slot=t)
        own.append(g)
    flat = [t for s in slots for t in uses[s]]
    part = dict(zip(flat, O.param_shift_grad(n, own, np.array(th), obs, slots=flat)))
    return np.array([sum(part[t] for t in uses[s]) for s in slots])


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_tile_items_vs_oracle(dt, graph):
    items = [item(n, k) for k, n in enumerate((12, 11, 13, 12, 4, 14))]
    b = Batch()
    b.set_graph(graph)
    for n, gates, theta, obs in items:
        b.add(Circuit.from_records(n, gates), Observable(n, obs), theta)
    for rep in range(3):
        e, g = b.run(dt)
        for i, (n, gates, theta, obs) in enumerate(items):
            scale = sum(abs(c) for c, _ in obs)
            assert abs(e[i] - O.energy(n, gates, theta, obs)) <= TOL[dt] * scale, (rep, i, n)
            slots = [0, 1, n // 2, n, len(theta) - 1]
            ref = shift_rule(n, gates, theta, obs, slots)
            assert np.max(np.abs(g[i][slots] - ref)) <= TOL[dt] * scale, (rep, i, n)
        if rep == 0:  # the same structure with other parameters
            items = [(n, gates, theta[::-1].copy(), obs) for n, gates, theta, obs in items]
            for i, it in enumerate(items):
                b.set_theta(i, it[2])
