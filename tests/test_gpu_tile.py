"""Tile passes (specialised kernels from 14 qubits on) where they can go
wrong: the smallest state (4 cosets of a tile), every gate kind with shared
parameters, rotations by multiples of pi (the tangent of the unnormalised form
is largest there), circuits with only one kind of rotation (many pending
factors, none of the diagonal gates that apply them), more gates and gradient
terms than one pass takes, and the qubit counts around the change of the
complex64 tile.  Against the CPU oracle, or above 20 qubits against the
interpreted kernels, with the tolerances of the other kernel forms."""
import numpy as np
import pytest

import synth
from oracle import grad as ogr, hamiltonian as oham, statevector as osv
from paper_2402_11878_amd import _lib, ansatz, hamiltonians as lham

from gpu_util import Dev, oracle_gates, rel_err, say, tol_energy
from test_host import random_circuit

pytestmark = pytest.mark.gpu

DT = {"c64": _lib.VQE_C64, "c128": _lib.VQE_C128}
AMP_TOL = {_lib.VQE_C64: 2e-5, _lib.VQE_C128: 1e-12}
GRAD_TOL = {_lib.VQE_C64: 1e-4, _lib.VQE_C128: 1e-9}
FORM_E_TOL = {_lib.VQE_C64: 1e-5, _lib.VQE_C128: 1e-12}
FORM_G_TOL = {_lib.VQE_C64: 1e-4, _lib.VQE_C128: 1e-11}


@pytest.fixture(autouse=True)
def _specialised():
    prev = _lib.vqe_set_specialize(_lib.SPECIALIZE_ALWAYS)
    yield
    _lib.vqe_set_specialize(prev)


def _circuit(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "random":  # every plain gate, parameters shared by several gates
        arr, P = random_circuit(n, 120, seed)
        arr["param_index"] %= np.int32(max(P // 2, 1))
        arr["param_index"][arr["kind"] > 2] = -1
        return arr, int(arr["param_index"].max()) + 1
    if kind == "excitation":
        arr, P = ansatz.excitations(n, 2)
        rot = ansatz.layered(n, 1)
        rot["param_index"][rot["param_index"] >= 0] += P
        return np.concatenate([arr, rot]), P + 2 * n
    if kind == "deep":  # more than 256 gates and 128 gradient terms in reach of the first window
        return ansatz.layered(n, 9), 18 * n
    g, p = [], 0
    gate = {"ry": 0, "rx": 2}[kind]
    for _ in range(4):
        for q in rng.permutation(n):
            g.append((gate, int(q), 0, p, 0.0))
            p += 1
        for q in range(0, n - 1, 2):
            g.append((5, q, q + 1, -1, 0.0))
    return ansatz.gates_array(g), p


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("n,kind,ckpt", [(14, "random", 0), (15, "random", 2), (14, "ry", 1), (14, "rx", 0),
                                         (14, "excitation", 1), (14, "deep", 0)])
def test_tile_passes_against_oracle(n, kind, ckpt, dt):
    dtype = DT[dt]
    arr, P = _circuit(kind, n, 5)
    rng = np.random.default_rng(6)
    th = rng.uniform(-4 * np.pi, 4 * np.pi, P)
    th[::3] = np.pi * rng.integers(-4, 5, size=len(th[::3]))
    H = {}
    for _ in range(20):
        s = tuple(rng.choice(list("IXYZ"), size=n, p=[0.4, 0.2, 0.2, 0.2]))
        H[s] = H.get(s, 0.0) + float(rng.normal())
    x, z, w = oham.to_masks(H)
    og = oracle_gates(arr)
    say(f"case tile n={n} {kind} {dt}")
    E_ref, g_ref = ogr.adjoint(n, og, th, H)
    h, c = _lib.vqe_hamiltonian_create(n, x, z, w), _lib.vqe_circuit_create(n, arr)
    s, l = Dev(n, dtype), Dev(n, dtype)
    cks = [Dev(n, dtype) for _ in range(ckpt)]
    try:
        _lib.vqe_state_set_basis(s.h, 0)
        _lib.vqe_apply_circuit(s.h, c, th)
        assert np.max(np.abs(s.read() - osv.run(n, og, th))) <= AMP_TOL[dtype]
        E, g = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=[d.h for d in cks])
        assert rel_err(E, E_ref) <= tol_energy(dtype)
        assert np.max(np.abs(g - g_ref)) / max(np.max(np.abs(g_ref)), 1.0) <= GRAD_TOL[dtype]
        back = s.read()  # the reverse sweep ends at the reference state
        back[0] -= 1
        assert np.max(np.abs(back)) <= AMP_TOL[dtype] * 10
        E2, g2 = _lib.vqe_energy_grad(s.h, l.h, c, th, h, ckpt=[d.h for d in cks], chunk_passes=1)
        assert E2 == E and np.array_equal(g2, g)  # fixed reduction order
    finally:
        for d in [s, l] + cks:
            d.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)


@pytest.mark.parametrize("n", [22, 23])
def test_tile_shapes_against_interpreted(n):
    """complex64 tiles of 12 (22 qubits) and 13 qubits (23), from a state that is no basis state."""
    arr = ansatz.layered(n, 3)
    th = synth.theta(n, 6 * n)
    x, z, w = lham.hubbard(11, synth.chain_bonds(11), 1.0, 4.0)
    c, h = _lib.vqe_circuit_create(n, arr), _lib.vqe_hamiltonian_create(n, x, z, w)
    s, l = Dev(n, _lib.VQE_C64), Dev(n, _lib.VQE_C64)
    say(f"case tile shapes n={n}")
    try:
        out = []
        for mode in (_lib.SPECIALIZE_ALWAYS, _lib.SPECIALIZE_NEVER):
            _lib.vqe_set_specialize(mode)
            E, g = _lib.vqe_energy_grad(s.h, l.h, c, th, h)
            _lib.vqe_state_set_basis(s.h, (1 << n) - 3)
            _lib.vqe_apply_circuit(s.h, c, th)
            _lib.vqe_apply_circuit(s.h, c, th[::-1].copy())
            out.append((E, g, s.t.cpu().numpy()))
        (E, g, a), (Ei, gi, ai) = out
        assert rel_err(E, Ei) <= FORM_E_TOL[_lib.VQE_C64]
        assert np.max(np.abs(g - gi)) / max(np.max(np.abs(gi)), 1.0) <= FORM_G_TOL[_lib.VQE_C64]
        assert np.max(np.abs(a - ai)) <= AMP_TOL[_lib.VQE_C64]
    finally:
        s.free(), l.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)
