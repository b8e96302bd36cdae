"""The planner's own time grows with the circuit, not with a power of it: deep
circuits on few qubits put all of their ops into one pass."""
import time

import numpy as np
import pytest

from paper_2011_13524_amd import Circuit, Plan
from paper_2011_13524_amd import workloads as W


def plan_seconds(n, gates, dt):
    c = Circuit.from_records(n, gates)
    best = 1e9
    for _ in range(3):
        t = time.perf_counter()
        Plan(c, dt)
        best = min(best, time.perf_counter() - t)
    return best


def phases(n, count):
    rng = np.random.default_rng(n)
    g = [{"op": "h", "q": [q]} for q in range(n)]
    for _ in range(count):  # controlled phases: all of them commute
        a, b = (int(x) for x in rng.permutation(n)[:2])
        g.append({"op": "dense", "q": [a], "mat": np.diag([1.0, np.exp(1j * rng.uniform(0, 6))]), "controls": [b],
                  "ctrl_vals": [1]})
    return g


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [9, 10, 11, 12, 13])
def test_layers(n, dt):
    # 16 times the layers: 16 times the time, with room for a busy machine (a
    # quadratic planner takes 256 times, one cubic in the ops of a pass 1200)
    short = plan_seconds(n, W.layered_rx_rz_cnot(n, 10, seed_key=(1,)), dt)
    assert plan_seconds(n, W.layered_rx_rz_cnot(n, 160, seed_key=(1,)), dt) <= 80 * short


@pytest.mark.parametrize("n", [10, 12])
def test_commuting_gates(n):
    short = plan_seconds(n, phases(n, 250), "c64")
    assert plan_seconds(n, phases(n, 4000), "c64") <= 80 * short
