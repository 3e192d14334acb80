"""Batch programs (the interpreter of small and mid-size states) where they can
go wrong: the smallest states (fewer qubits than a wave has amplitudes for),
the changes of size (10 / 11 qubits, the largest small state, the first mid-size
one), more gates on few qubits than a stage's block holds, every gate kind with
shared parameters, rotations by multiples of pi, excitations, checkpoints,
Hamiltonians of few terms and of several blocks, with real and complex
coefficients.  Against the CPU oracle with the tolerances of the other kernel
forms, through the batch and the single evaluation, which returns |0...0>."""
import numpy as np
import pytest

from oracle import grad as ogr, hamiltonian as oham
from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, oracle_gates, say
from test_host import random_circuit

pytestmark = pytest.mark.gpu

DT = {"c64": _lib.VQE_C64, "c128": _lib.VQE_C128}
E_TOL = {_lib.VQE_C64: 1e-5, _lib.VQE_C128: 1e-10}
GRAD_TOL = {_lib.VQE_C64: 1e-4, _lib.VQE_C128: 1e-9}
AMP_TOL = {_lib.VQE_C64: 2e-5, _lib.VQE_C128: 1e-12}


def _circuit(kind, n):
    if kind == "random":
        arr, P = random_circuit(n, 30 * n, 11)
        arr["param_index"] %= np.int32(max(P // 2, 1))
        arr["param_index"][arr["kind"] > 2] = -1
        return arr, int(arr["param_index"].max()) + 1
    if kind == "deep":  # rotations of one qubit after another: many rows per stage, more than a block
        g, p = [], 0
        for k in range(150):
            for q in range(n):
                g.append(((0, 1, 2)[(k + q) % 3] if k % 5 else 0, q, 0, p % 40, 0.0))
                p += 1
            if n > 1:
                g.append((5, k % n, (k + 1) % n, -1, 0.0))
        return ansatz.gates_array(g), 40
    if kind == "cnot":  # nothing to sum or turn: stages of CNOTs and X alone
        g = [(0, q, 0, q, 0.0) for q in range(n)]
        g += [(5, q, (q + 1) % n, -1, 0.0) for _ in range(3) for q in range(n)]
        return ansatz.gates_array(g), n
    if kind == "none":
        return ansatz.gates_array([]), 0
    arr, P = ansatz.excitations(n, 2)
    rot = ansatz.layered(n, 1)
    rot["param_index"][rot["param_index"] >= 0] += P
    return np.concatenate([rot, arr, rot]), P + 2 * n


def _hamiltonian(n, terms, seed):
    rng = np.random.default_rng(seed)
    H = {}
    for _ in range(terms):
        s = tuple(rng.choice(list("IXYZ"), size=n, p=[0.4, 0.2, 0.2, 0.2]))
        H[s] = H.get(s, 0.0) + float(rng.normal())
    return H


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n,kind,terms,ckpt", [(1, "random", 3, 0), (3, "deep", 20, 2), (4, "deep", 40, 0), (4, "none", 5, 0),
                                               (6, "excitation", 60, 1), (10, "random", 600, 2), (11, "cnot", 30, 1),
                                               (11, "excitation", 30, 3), (12, "random", 30, 0), (13, "random", 20, 1),
                                               (13, "none", 20, 0), (14, "random", 20, 0), (15, "excitation", 15, 0),
                                               (14, "deep", 20, 2), (17, "random", 10, 3), (14, "none", 10, 1)])
def test_programs_against_oracle(n, kind, terms, ckpt, dt):
    dtype = DT[dt]
    arr, P = _circuit(kind, n)
    rng = np.random.default_rng(n)
    th = rng.uniform(-4 * np.pi, 4 * np.pi, P)
    th[::3] = np.pi * rng.integers(-4, 5, size=len(th[::3]))
    H = _hamiltonian(n, terms, n + 1)
    x, z, w = oham.to_masks(H)
    E_ref, g_ref = ogr.adjoint(n, oracle_gates(arr), th, H)
    # rounding errors of E and of a gradient term grow with |H psi| ~ |w|
    scale = max(abs(E_ref), float(np.linalg.norm(w)), 1.0)
    gscale = max(float(np.abs(g_ref).max()) if P else 1.0, scale)
    import torch
    say(f"case program n={n} {kind} terms={terms} {dt}")
    h, c = _lib.vqe_hamiltonian_create(n, x, z, w), _lib.vqe_circuit_create(n, arr)
    b = _lib.vqe_batch_create(dtype, torch.cuda.current_stream().cuda_stream)
    held = []
    try:
        (E, g), (E2, g2) = _lib.vqe_batch_energy_grad(b, [(c, h, th)] * 2)
        assert abs(E - E_ref) <= E_TOL[dtype] * scale
        assert P == 0 or np.abs(np.asarray(g) - g_ref).max() <= GRAD_TOL[dtype] * gscale
        assert E == E2 and np.array_equal(g, g2)
        s, l = Dev(n, dtype), Dev(n, dtype)
        cks = [Dev(n, dtype) for _ in range(ckpt)]
        held = [s, l] + cks
        E1, g1 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=[k.h for k in cks])
        assert abs(E1 - E_ref) <= E_TOL[dtype] * scale
        assert P == 0 or np.abs(np.asarray(g1) - g_ref).max() <= GRAD_TOL[dtype] * gscale
        E3, g3 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=[k.h for k in cks], chunk_passes=1)
        assert E3 == E1 and np.array_equal(g3, g1)  # submission in chunks changes nothing
        if ckpt:  # nor do checkpoints, up to rounding
            E4, g4 = _lib.vqe_energy_grad(s.h, l.h, c, th, h)
            assert E4 == E1 and (P == 0 or np.abs(g4 - g1).max() <= GRAD_TOL[dtype] * gscale)
        back = s.read()
        back[0] -= 1
        assert np.abs(back).max() <= AMP_TOL[dtype] * 10
    finally:
        for d in held:
            d.free()
        _lib.vqe_batch_free(b)
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)
