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


def test_rotations_give_their_matrix_back():
    # complex128: a matrix runs as a rotation between diagonals only where the rounded
    # factors stand for it to half a unit in the last place of 1
    L = Q.lib()
    runs = getattr(L, "_ZN3qsv16runs_as_rotationEPKNS_2cdEb")
    runs.restype = ctypes.c_bool
    runs.argtypes = [ctypes.c_void_p, ctypes.c_bool]
    split = getattr(L, "_ZN3qsv19unitary_to_rotationEPKNS_2cdEPS0_")
    split.restype = None
    split.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    rng = np.random.default_rng(5)
    h = np.array([[1, 1], [1, -1]]) * np.sqrt(0.5)  # (the named gate's entries)
    y = np.array([[0, -1j], [1j, 0]])
    assert runs(np.ascontiguousarray(h, dtype=np.complex128).ctypes.data, False)
    taken = 0
    for u in [h, y] + [W.haar_unitary(rng, 2) for _ in range(200)]:
        u = np.ascontiguousarray(u, dtype=np.complex128)
        assert runs(u.ctypes.data, True)
        if not runs(u.ctypes.data, False):
            continue
        taken += 1
        o = np.zeros(6, dtype=np.complex128)
        split(u.ctypes.data, o.ctypes.data)
        a, b = np.longdouble(o[2].real), np.longdouble(o[2].imag)
        m = np.array([[1 + a * b, a * (2 + a * b)], [b, 1 + a * b]])
        got = o[4:, None].astype(np.clongdouble) * m * o[None, :2].astype(np.clongdouble)
        assert np.max(np.abs(got - u.astype(np.clongdouble))) <= 1.3e-16
    assert 2 <= taken < 100  # (the named gates and few others)
