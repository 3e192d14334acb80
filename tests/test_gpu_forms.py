"""The kernel form (vqe_set_specialize) is process-wide and may be changed by any
thread at any time: an evaluation reads it once and keeps to one plan.
Checkpoints and chunked submission in every form."""
import threading

import numpy as np
import pytest

from oracle import grad as ogr, hamiltonian as oham
from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, oracle_gates, rel_err, say

pytestmark = pytest.mark.gpu

DT = {"c64": _lib.VQE_C64, "c128": _lib.VQE_C128}
FORMS = {"never": _lib.SPECIALIZE_NEVER, "auto": _lib.SPECIALIZE_AUTO, "always": _lib.SPECIALIZE_ALWAYS}
E_TOL = {_lib.VQE_C64: 1e-5, _lib.VQE_C128: 1e-10}
GRAD_TOL = {_lib.VQE_C64: 1e-4, _lib.VQE_C128: 1e-9}


def _problem(n, layers, seed):
    rng = np.random.default_rng(seed)
    x = np.array([0, 1, 6, 1 << (n - 1), 3 << (n - 2), 5], np.uint64)
    z = rng.choice(1 << n, size=len(x), replace=False).astype(np.uint64)
    w = rng.normal(size=len(x))
    arr = ansatz.layered(n, layers)
    th = rng.uniform(-np.pi, np.pi, size=2 * n * layers)
    ref = ogr.adjoint(n, oracle_gates(arr), th, oham.from_masks(n, x, z, w))
    return _lib.vqe_circuit_create(n, arr), _lib.vqe_hamiltonian_create(n, x, z, w), th, ref


@pytest.mark.parametrize("n,dt", [(12, "c64"), (14, "c64"), (14, "c128")])
def test_form_changed_by_another_thread(n, dt):
    """Evaluations while another thread goes through the forms: every one
    gives the gradient, by whichever form it began with."""
    dtype = DT[dt]
    say(f"case forms race n={n} {dt}")
    c, h, th, (E_ref, g_ref) = _problem(n, 3, n)
    d = [Dev(n, dtype) for _ in range(3)]
    old = _lib.vqe_set_specialize(_lib.SPECIALIZE_AUTO)
    stop = threading.Event()

    def flip():
        while not stop.is_set():
            for f in (_lib.SPECIALIZE_ALWAYS, _lib.SPECIALIZE_NEVER, _lib.SPECIALIZE_AUTO, _lib.SPECIALIZE_NEVER):
                _lib.vqe_set_specialize(f)

    def check(E, g):
        assert rel_err(E, E_ref) <= E_TOL[dtype]
        assert np.max(np.abs(g - g_ref)) / max(np.max(np.abs(g_ref)), 1) <= GRAD_TOL[dtype]

    try:
        for f in FORMS.values():  # compiles the kernels of every form
            _lib.vqe_set_specialize(f)
            check(*_lib.vqe_energy_grad(d[0].h, d[1].h, c, th, h))
        t = threading.Thread(target=flip)
        t.start()
        try:
            for k in range(200):
                check(*_lib.vqe_energy_grad(d[0].h, d[1].h, c, th, h, ckpt=[d[2].h] if k % 2 else []))
                _lib.vqe_state_set_basis(d[0].h, 0)
                _lib.vqe_apply_circuit(d[0].h, c, th)
                assert rel_err(_lib.vqe_expect_pauli(d[0].h, h)[0], E_ref) <= E_TOL[dtype]
        finally:
            stop.set()
            t.join()
    finally:
        _lib.vqe_set_specialize(old)
        for s in d:
            s.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("form,n", [("never", 13), ("never", 14), ("always", 11), ("always", 13), ("always", 14),
                                    ("auto", 13), ("auto", 15)])
def test_checkpoints_and_chunks(form, n, dt):
    """Checkpoints and chunked submission in every kernel form: interpreted and
    specialised windows, tile passes, one launch, mid-size passes.  Chunks give
    the bits of the unchunked sweep, checkpoints the energy's bits and the
    gradient up to the rounding of un-applying fewer gates."""
    dtype = DT[dt]
    say(f"case forms checkpoints {form} n={n} {dt}")
    c, h, th, (E_ref, g_ref) = _problem(n, 5, n)
    d = [Dev(n, dtype) for _ in range(5)]
    s, l, cks = d[0], d[1], d[2:]
    old = _lib.vqe_set_specialize(FORMS[form])
    try:
        E0, g0 = _lib.vqe_energy_grad(s.h, l.h, c, th, h)
        assert rel_err(E0, E_ref) <= E_TOL[dtype]
        assert np.max(np.abs(g0 - g_ref)) / max(np.max(np.abs(g_ref)), 1) <= GRAD_TOL[dtype]
        passes = _lib.vqe_circuit_info(c)[1]
        for chunk in (1, 2, 3, passes, passes + 5):
            E1, g1 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, chunk_passes=chunk)
            assert E1 == E0 and np.array_equal(g1, g0), chunk
        for k in (1, 3):
            ck = [b.h for b in cks[:k]]
            E1, g1 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=ck)
            assert rel_err(E1, E0) <= E_TOL[dtype]
            assert np.max(np.abs(g1 - g_ref)) / max(np.max(np.abs(g_ref)), 1) <= GRAD_TOL[dtype]
            E2, g2 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=ck, chunk_passes=2)
            assert E2 == E1 and np.array_equal(g2, g1)
    finally:
        _lib.vqe_set_specialize(old)
        for b in d:
            b.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("form,n", [("never", 16), ("auto", 16), ("auto", 20)])
def test_chunks_of_h_psi(form, n, dt):
    """chunk_passes over a Hamiltonian of several window passes, waiting within
    H psi too: the bits of the unchunked evaluation."""
    dtype = DT[dt]
    say(f"case forms chunks of H psi {form} n={n} {dt}")
    rng = np.random.default_rng(n)
    x = np.array([0] + [3 << a for a in range(n - 1)] + [(1 << a) | (1 << b) for a in range(n) for b in range(a)],
                 np.uint64)
    h = _lib.vqe_hamiltonian_create(n, x, rng.integers(0, 1 << n, size=len(x)).astype(np.uint64),
                                    rng.normal(size=len(x)))
    m = len(_lib.vqe_hamiltonian_plan(h))
    assert m > 2
    c = _lib.vqe_circuit_create(n, ansatz.layered(n, 2))
    th = rng.uniform(-np.pi, np.pi, size=4 * n)
    s, l, ck = Dev(n, dtype), Dev(n, dtype), Dev(n, dtype)
    old = _lib.vqe_set_specialize(FORMS[form])
    try:
        for ckpt in ([], [ck.h]):
            E0, g0 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=ckpt)
            for chunk in (1, 2, m, 100):
                E1, g1 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=ckpt, chunk_passes=chunk)
                assert E1 == E0 and np.array_equal(g1, g0), chunk
    finally:
        _lib.vqe_set_specialize(old)
        for b in (s, l, ck):
            b.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)
