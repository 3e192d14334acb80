"""Specialised window kernels work in place: passes of X and CNOT gates alone,
which only exchange amplitudes, against the oracle (states below the tile
passes, both dtypes).  Such gates are exact, so the tolerance is that of the one
layer of rotations."""
import numpy as np
import pytest

from oracle import statevector as osv
from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, oracle_gates, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,tol", [(_lib.VQE_C64, 2e-6), (_lib.VQE_C128, 1e-14)])
@pytest.mark.parametrize("n", [6, 10, 13])
def test_renames_alone_in_place(n, dt, tol):
    g = [(0, q, 0, q, 0.0) for q in range(n)]
    rng = np.random.default_rng(n)
    for _ in range(12):
        g += [(4, int(rng.integers(n)), 0, -1, 0.0)]
        for _ in range(6):
            a, b = rng.choice(n, 2, replace=False)
            g.append((5, int(a), int(b), -1, 0.0))
    arr = ansatz.gates_array(g)
    th = rng.uniform(-3, 3, n)
    say(f"case in place n={n} dtype={dt}")
    prev = _lib.vqe_set_specialize(_lib.SPECIALIZE_ALWAYS)
    c, h = _lib.vqe_circuit_create(n, arr), _lib.vqe_hamiltonian_create(n, [0, 1], [1, 0], [1.0, 0.5])
    s, l = Dev(n, dt), Dev(n, dt)
    try:
        _lib.vqe_state_set_basis(s.h, 0)
        _lib.vqe_apply_circuit(s.h, c, th)
        assert np.abs(s.read() - osv.run(n, oracle_gates(arr), th)).max() <= tol
        _lib.vqe_energy_grad(s.h, l.h, c, th, h)
        back = np.abs(s.read())  # the reference state up to a sign
        back[0] -= 1
        assert np.abs(back).max() <= tol
    finally:
        _lib.vqe_set_specialize(prev)
        s.free()
        l.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)
