"""One observable used by two threads on two streams: the tables that expectations use
stay in place when another thread's first lambda pass makes its own, and the other
way round.
"""
import threading

import numpy as np
import pytest

from paper_2011_13524_amd import Observable, State, apply_observable, expectation
from paper_2011_13524_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("first", ["expectation", "lambda"])
def test_first_calls_beside_running_ones(dt, first):
    import torch
    n = 15
    terms = W.random_pauli_observable(n, 120, (1, 5), seed_key=(n, 2)) + [(0.3, [])]
    rng = np.random.default_rng(n)
    v = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    v /= np.linalg.norm(v)
    streams = [torch.cuda.Stream() for _ in range(2)]
    a, b, lam, ref = (State(n, dt, stream=s) for s in (streams[0], streams[1], streams[1], streams[0]))
    a.load(v)
    b.load(v)
    fresh = Observable(n, terms)
    want = expectation(a, fresh)
    apply_observable(a, Observable(n, terms), ref)
    want_lam = ref.store()
    for _ in range(4):
        o = Observable(n, terms)
        got, lams = [], []

        def energies():
            for _ in range(30):
                got.append(expectation(a, o))

        def lambdas():
            for _ in range(10):
                apply_observable(b, o, lam)
                lams.append(lam.store())

        (energies if first == "expectation" else lambdas)()  # (its tables are there)
        threads = [threading.Thread(target=f) for f in (energies, lambdas)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert all(e == want for e in got)
        assert all(np.array_equal(x, want_lam) for x in lams)
