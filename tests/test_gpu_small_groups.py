"""H psi of small states over X groups of 1 to 6 terms, summed term by term, next
to ones summed by buckets (also of more terms than a bucket counts), with real and
complex coefficients, against the CPU oracle with the tolerances of the other
tests of the batch programs."""
import numpy as np
import pytest

from oracle import grad as ogr, hamiltonian as oham
from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, oracle_gates, rel_err, say

pytestmark = pytest.mark.gpu

DT = {"c64": _lib.VQE_C64, "c128": _lib.VQE_C128}
E_TOL = {_lib.VQE_C64: 1e-5, _lib.VQE_C128: 1e-10}
GRAD_TOL = {_lib.VQE_C64: 1e-4, _lib.VQE_C128: 1e-9}


def _masks(n, sizes, real, seed):
    rng = np.random.default_rng(seed)
    x, z = [], []
    for m, k in zip(rng.choice(1 << n, size=len(sizes), replace=False), sizes):
        zs = rng.permutation(1 << n)
        if real:
            zs = [v for v in zs if bin(int(v) & int(m)).count("1") % 2 == 0]
        x += [m] * min(k, len(zs))
        z += list(zs[:k])
    return np.array(x, np.uint64), np.array(z, np.uint64), rng.normal(size=len(x))


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("real", [True, False])
@pytest.mark.parametrize("n", [3, 4, 10, 11, 12, 13])
def test_group_sizes(n, real, dt):
    dtype = DT[dt]
    if n > _lib.BATCH_MAX_QUBITS[dtype]:
        pytest.skip("not a small state")
    say(f"case small groups n={n} real={real} {dt}")
    sizes = ([1, 2, 3, 4, 5, 6, 1][: 1 << n] if n < 8 else [1, 2, 3, 4, 5, 6, 30, 1, 600, 4, 3, 7] * 2)
    arr, th = ansatz.layered(n, 2), np.random.default_rng(n).uniform(-3, 3, size=4 * n)
    d = [Dev(n, dtype), Dev(n, dtype)]
    c = _lib.vqe_circuit_create(n, arr)
    try:
        for sz in (sizes, [1], [2], [4, 4]):
            x, z, w = _masks(n, sz, real, n + len(sz))
            h = _lib.vqe_hamiltonian_create(n, x, z, w)
            E, g = _lib.vqe_energy_grad(d[0].h, d[1].h, c, th, h)
            _lib.vqe_hamiltonian_free(h)
            E_ref, g_ref = ogr.adjoint(n, oracle_gates(arr), th, oham.from_masks(n, x, z, w))
            assert rel_err(E, E_ref) <= E_TOL[dtype], sz
            assert np.max(np.abs(g - g_ref)) / max(np.max(np.abs(g_ref)), 1) <= GRAD_TOL[dtype], sz
    finally:
        for s in d:
            s.free()
        _lib.vqe_circuit_free(c)
