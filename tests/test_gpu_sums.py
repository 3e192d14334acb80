"""Partial sums of the gradient terms in complex64: a thread of a batch program
holds 16 amplitudes per vector, and the terms of their pairs are summed in 64
bits, as the sums over threads are.

The inputs make every float operation exact except sums of more than two pairs
in 32 bits.  RY(pi/2) on every qubit gives all amplitudes 2^(-n/2) (n even; the
rotations of a stage wait together, four factors cos(pi/4) make 1/4), and
H = Z_b + B Z_b Z_c with B = 2^23 gives lam = +-(B +- 1) psi, all 24 bits of the
type.  The term of B cancels over c, dE/dtheta of RY(theta = 0) on b is -1:
a sum of three equal pairs in 32 bits already loses its last bit, which is the
answer.  With Y_b in place of Z_b the same holds for RZ(theta = 0), with +1."""
import numpy as np
import pytest

from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("probe", ["RY", "RZ"])
@pytest.mark.parametrize("form,n", [("batch", 10), ("batch", 12), ("batch", 16), ("single", 12), ("single", 16)])
def test_terms_of_pairs_are_summed_in_64_bits(form, n, probe):
    say(f"case sums {form} n={n} {probe}")
    g = [(0, q, 0, -1, np.pi / 2) for q in range(n)]
    g += [(0 if probe == "RY" else 1, q, 0, q, 0.0) for q in range(n)]
    c = _lib.vqe_circuit_create(n, ansatz.gates_array(g))
    th = np.zeros(n)
    want = -1.0 if probe == "RY" else 1.0
    d = [Dev(n, _lib.VQE_C64), Dev(n, _lib.VQE_C64)] if form == "single" else []
    b = _lib.vqe_batch_create(_lib.VQE_C64, None) if form == "batch" else None
    try:
        for q in range(n):
            for o in (k for k in range(n) if k != q):
                x = 0 if probe == "RY" else 1 << q
                masks = np.array([x, x], np.uint64), np.array([1 << q, (1 << q) | (1 << o)], np.uint64)
                h = _lib.vqe_hamiltonian_create(n, *masks, np.array([1.0, 2.0 ** 23]))
                if b is not None:
                    _, gr = _lib.vqe_batch_energy_grad(b, [(c, h, th)])[0]
                else:
                    _, gr = _lib.vqe_energy_grad(d[0].h, d[1].h, c, th, h)
                _lib.vqe_hamiltonian_free(h)
                assert gr[q] == want, (q, o, gr[q])
    finally:
        for s in d:
            s.free()
        if b is not None:
            _lib.vqe_batch_free(b)
        _lib.vqe_circuit_free(c)
