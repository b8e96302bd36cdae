"""The planner's test that decides whether a one-qubit matrix becomes a rotation
between diagonals: unitary up to a real factor, at every size of the factor."""
import ctypes

import numpy as np
import pytest

import paper_2011_13524_amd as Q
from paper_2011_13524_amd import workloads as W


@pytest.mark.parametrize("tol", [2e-15, 1e-9])
@pytest.mark.parametrize("scale", [1.0, 1e-100, 1e100, 1e-161, 3e-162, 1e-170, 1e160, 1e300])
def test_matrices_off_unitary_are_told_at_every_scale(tol, scale):
    f = getattr(Q.lib(), "_ZN3qsv11is_unitary2EPKNS_2cdEd")
    f.restype = ctypes.c_bool
    f.argtypes = [ctypes.c_void_p, ctypes.c_double]

    def unitary(m):
        m = np.ascontiguousarray(m, dtype=np.complex128)
        return f(m.ctypes.data, tol)

    u = W.haar_unitary(np.random.default_rng(3), 2)
    assert not unitary(scale * np.array([[1.0, 0.01], [0.0, 1.0]]))
    assert not unitary(scale * (u + 0.01 * np.eye(2)))
    if 1e-120 < scale < 1e120:  # (squares in range)
        assert unitary(scale * u) or tol < 1e-14
        assert unitary(scale * np.diag([1.0, -1.0]))
