"""vqe_circuit_prepare takes the planning of the batch programs out of the first
evaluation: on deep circuits, where planning takes a few milliseconds."""
import time

import numpy as np
import pytest

from paper_2402_11878_amd import _lib, ansatz

from gpu_util import Dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,n,layers", [("single", 10, 300), ("single", 15, 100), ("batch", 10, 300), ("batch", 15, 100)])
def test_first_evaluation_after_prepare(form, n, layers):
    """The first evaluation of a prepared circuit takes little longer than the
    next ones (the best of four circuits; buffers are there from another of the
    same size): 1.01 times as long, 1.38 where planning is left to it."""
    say(f"case prepare {form} n={n} layers={layers}")
    arr = ansatz.layered(n, layers)
    th = np.random.default_rng(n).uniform(-3, 3, size=2 * n * layers)
    h = _lib.vqe_hamiltonian_create(n, np.array([1, 3], np.uint64), np.array([1, 0], np.uint64), np.array([1.0, 0.5]))
    d = [Dev(n, _lib.VQE_C64), Dev(n, _lib.VQE_C64)] if form == "single" else []
    b = _lib.vqe_batch_create(_lib.VQE_C64, None) if form == "batch" else None

    def run(c):
        t = time.perf_counter()
        if b is not None:
            _lib.vqe_batch_energy_grad(b, [(c, h, th)])
        else:
            _lib.vqe_energy_grad(d[0].h, d[1].h, c, th, h)
        return time.perf_counter() - t

    ratios = []
    try:
        for k in range(5):
            c = _lib.vqe_circuit_create(n, arr)
            _lib.vqe_circuit_prepare(c, _lib.VQE_C64)
            first = run(c)
            later = min(run(c) for _ in range(5))
            _lib.vqe_circuit_free(c)
            say(f"  first {first * 1e6:.0f} us, later {later * 1e6:.0f} us")
            if k:
                ratios.append(first / later)
        assert min(ratios) <= 1.2, ratios
    finally:
        for s in d:
            s.free()
        if b is not None:
            _lib.vqe_batch_free(b)
        _lib.vqe_hamiltonian_free(h)
