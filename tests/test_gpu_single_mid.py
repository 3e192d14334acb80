"""Single evaluations above the LDS limit and below the specialised sizes: lam =
H psi runs by window passes or as one sweep over tiles, and the trace counts the
bytes that a pass must move (the first forward pass stages |0...0> and only
writes).  Energies and gradients against the oracle."""
import numpy as np
import pytest

from oracle import grad as ogr, hamiltonian as oham
from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, oracle_gates, rel_err, say

pytestmark = pytest.mark.gpu

DT = {"c64": _lib.VQE_C64, "c128": _lib.VQE_C128}
E_TOL = {_lib.VQE_C64: 1e-5, _lib.VQE_C128: 1e-10}
GRAD_TOL = {_lib.VQE_C64: 1e-4, _lib.VQE_C128: 1e-9}


def _masks(kind, n):
    """tile, wide: two 10-bit X masks that two windows hold, where the plan of large
    states takes tiles: so do few terms per group, many take windows; nocover: a
    mask that no window holds; window: one window."""
    rng = np.random.default_rng(n)
    x = {"tile": [0, 0x3ff << 3, 0x3ff << (n - 10)], "wide": [0, 0x3ff << 3, 0x3ff << (n - 10)], "nocover": [0, (1 << n) - 1, 5, 0x3ff << (n - 10)],
         "window": [0, 1, 6, 1 << 11]}[kind]
    x = np.repeat(np.array(x, np.uint64), 7 if kind == "wide" else 3)
    z = rng.choice(1 << n, size=len(x), replace=False).astype(np.uint64)
    return x, z, rng.normal(size=len(x))


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [14, 16])
@pytest.mark.parametrize("kind", ["tile", "wide", "nocover", "window"])
def test_form_and_traced_bytes(kind, n, dt):
    dtype = DT[dt]
    say(f"case single mid {kind} n={n} {dt}")
    x, z, w = _masks(kind, n)
    th = np.random.default_rng(3).uniform(-3, 3, size=2 * n * 2)
    arr = ansatz.layered(n, 2)
    h = _lib.vqe_hamiltonian_create(n, x, z, w)
    c = _lib.vqe_circuit_create(n, arr)
    s, l = Dev(n, dtype), Dev(n, dtype)
    S = (8 if dtype == _lib.VQE_C64 else 16) << n
    try:
        m = len(_lib.vqe_hamiltonian_plan(h))
        assert (m > 0) == (kind == "window")
        _lib.vqe_profile_enable(True)
        _lib.vqe_profile_reset()
        E, g = _lib.vqe_energy_grad(s.h, l.h, c, th, h)
        fwd, rev, hp = (_lib.vqe_profile_read(k) for k in (0, 1, 2))
        assert fwd[2] == (2 * fwd[0] - 1) * S
        assert rev[2] == 4 * rev[0] * S and rev[0] == fwd[0]
        D = len({int(v) >> 10 for v in x} - {0})
        m = 2 if kind == "wide" else m
        assert (hp[0], hp[2]) == ((m, (3 * m - 1) * S) if m else (1, (D + 2) * S))
        E_ref, g_ref = ogr.adjoint(n, oracle_gates(arr), th, oham.from_masks(n, x, z, w))
        assert rel_err(E, E_ref) <= E_TOL[dtype]
        assert np.max(np.abs(g - g_ref)) / max(np.max(np.abs(g_ref)), 1) <= GRAD_TOL[dtype]
    finally:
        _lib.vqe_profile_enable(False)
        _lib.vqe_profile_reset()
        s.free()
        l.free()
        _lib.vqe_circuit_free(c)
        _lib.vqe_hamiltonian_free(h)
