"""Window passes of H psi where they can go wrong: one coset (13 qubits, fewer
cosets than blocks), several per block, passes of more terms than LDS keeps, the
two register budgets of complex64 (blocks alone on a CU and in pairs), real and
complex coefficients.  The energy-only form counts one of each pair of patterns:
X masks on the lane, wave and register part of the window, alone and mixed.
Against the CPU oracle, above 16 qubits against one sweep per term."""
import numpy as np
import pytest

from oracle import statevector as osv
from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, oracle_gates, say

pytestmark = pytest.mark.gpu

DT = {"c64": _lib.VQE_C64, "c128": _lib.VQE_C128}
E_TOL = {_lib.VQE_C64: 1e-5, _lib.VQE_C128: 1e-12}
AMP_TOL = {_lib.VQE_C64: 2e-5, _lib.VQE_C128: 1e-12}


def _terms(n, real, many, seed):
    """Masks: one group per pair of bits of the first window and none, with z strings; many: > 512 terms of one pass."""
    rng = np.random.default_rng(seed)
    xs = [0, 1, 2, 3, 1 << 6, 1 << 7, 1 << 9, 1 << 10, 1 << 12, (1 << 12) | 1, (1 << 11) | (1 << 8), (1 << 5) | (1 << 4),
          3 << 10, 3 << 11]
    x, z = [], []
    for m in xs:
        for _ in range(64 if many else 6):
            zz = int(rng.integers(0, 1 << n))
            if many:  # 16 patterns in the window, so that its classes stay below a pass's limit
                zz &= ~((1 << 13) - 1) | 0x78
            if real and bin(zz & m).count("1") % 2:  # an odd number of Y: drop one
                zz &= ~(zz & m & -(zz & m))
            x.append(m)
            z.append(zz)
    _, keep = np.unique(np.array(x, dtype=np.uint64) << np.uint64(32) | np.array(z, dtype=np.uint64), return_index=True)
    x, z = np.array(x, np.uint64)[keep], np.array(z, np.uint64)[keep]
    return x, z, rng.normal(size=len(x))


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n,real,many", [(13, True, True), (13, False, False), (14, True, False), (15, True, True), (16, False, True)])
def test_window_passes_against_oracle(n, real, many, dt):
    dtype = DT[dt]
    x, z, w = _terms(n, real, many, n)
    arr = ansatz.layered(n, 2)
    th = np.random.default_rng(n).uniform(-3, 3, 4 * n)
    psi = osv.run(n, oracle_gates(arr), th)
    ref, b = np.zeros_like(psi), np.arange(1 << n, dtype=np.uint64)
    for xm, zm, wt in zip(x, z, w):  # i^(number of Y) X^x Z^z
        q = b ^ xm
        sign = 1 - 2 * (np.bitwise_count(q & zm).astype(np.int8) & 1)
        ref += wt * 1j ** bin(int(xm & zm)).count("1") * sign * psi[q]
    h, c = _lib.vqe_hamiltonian_create(n, x, z, w), _lib.vqe_circuit_create(n, arr)
    s, l = Dev(n, dtype), Dev(n, dtype)
    say(f"case hwin n={n} real={real} many={many} {dt}")
    scale = np.abs(w).sum()  # bound of |H|
    try:
        _lib.vqe_state_set_basis(s.h, 0)
        _lib.vqe_apply_circuit(s.h, c, th)
        e, _ = _lib.vqe_expect_pauli(s.h, h, _lib.EXPECT_GROUPED)
        el, _ = _lib.vqe_apply_hamiltonian(s.h, l.h, h)
        lam = l.read()
        E = float(np.vdot(psi, ref).real)
        assert abs(e - E) <= E_TOL[dtype] * scale and abs(el - E) <= E_TOL[dtype] * scale
        assert np.abs(lam - ref).max() <= AMP_TOL[dtype] * scale
    finally:
        s.free()
        l.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)


@pytest.mark.parametrize("dt,n", [("c64", 21), ("c64", 22), ("c128", 22)])
def test_window_passes_against_terms(n, dt):
    dtype = DT[dt]
    x, z, w = _terms(n, True, False, n)
    arr = ansatz.layered(n, 1)
    th = np.random.default_rng(n).uniform(-3, 3, 2 * n)
    h, c = _lib.vqe_hamiltonian_create(n, x, z, w), _lib.vqe_circuit_create(n, arr)
    s, l = Dev(n, dtype), Dev(n, dtype)
    say(f"case hwin terms n={n} {dt}")
    try:
        _lib.vqe_state_set_basis(s.h, 0)
        _lib.vqe_apply_circuit(s.h, c, th)
        E, _ = _lib.vqe_expect_pauli(s.h, h, _lib.EXPECT_PER_TERM)
        e, _ = _lib.vqe_expect_pauli(s.h, h, _lib.EXPECT_GROUPED)
        el, _ = _lib.vqe_apply_hamiltonian(s.h, l.h, h)
        scale = np.abs(w).sum()
        assert abs(e - E) <= E_TOL[dtype] * scale and abs(el - E) <= E_TOL[dtype] * scale
    finally:
        s.free()
        l.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)
