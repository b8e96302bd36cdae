"""Host-side tables of the reverse sweep that stay with a forward plan: which
circuits they are made for. No device is used; each case runs in a process of its
own, so that one that ends it is told from the others.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import ctypes, sys
import paper_2011_13524_amd as Q
dtype, paulis = sys.argv[1], [int(p) for p in sys.argv[2]]
f = getattr(Q.lib(), "_ZN3qsv13adjoint_cacheI%sEEPNS_8AdjCacheEP8qsv_planPK11qsv_circuit" % ("f" if dtype == "c64" else "d"))
f.restype = ctypes.c_void_p
f.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
for n in map(int, sys.argv[3:]):
    c = Q.Circuit.from_records(n, [{"op": "h", "q": [q]} for q in range(n)] +
                               [{"op": "pauli_rot", "q": list(range(len(paulis))), "paulis": paulis, "slot": 0},
                                {"op": "rx", "q": [n - 1], "slot": 1}])
    p = Q.Plan(c, dtype)
    print(n, "kept" if f(p.h, c.h) else "none", flush=True)
"""


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("paulis", ["33", "333", "31", "3"])
def test_tables_kept_with_a_plan(dtype, paulis):
    # a parametric Pauli string: tables from 9 qubits (register-resident sweeps), of
    # Z strings on two or more qubits (their value is a DynVal); otherwise none
    sizes = [3, 5, 8, 9, 11, 12, 13]
    r = subprocess.run([sys.executable, "-c", PROGRAM, dtype, paulis, *map(str, sizes)], cwd=ROOT, capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    z = len(paulis) > 1 and set(paulis) == {"3"}
    assert r.stdout.split("\n")[:-1] == ["%d %s" % (n, "kept" if n >= 9 and z else "none") for n in sizes]
