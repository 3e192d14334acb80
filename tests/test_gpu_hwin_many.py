"""H psi window passes with more than one coset per compute unit: two blocks on
each (complex64, with lam and energy only) and blocks that go on from coset to
coset (complex128), element by element against the same sums in 64 bits."""
import numpy as np
import pytest

from paper_2402_11878_amd import _lib

from gpu_util import Dev, say
from test_gpu_hwin import AMP_TOL, DT, E_TOL, _terms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("dt,n", [("c64", 22), ("c64", 23), ("c128", 22), ("c128", 23), ("c128", 24)])
def test_lam_and_energy(dt, n, many):
    import torch
    dtype = DT[dt]
    say(f"case hwin many n={n} {dt} terms={'many' if many else 'few'}")
    x, z, w = _terms(n, True, many, n)
    # a last mask on high qubits: a second pass, which reads lam
    x = np.append(x, np.uint64(3 << (n - 2)))
    z, w = np.append(z, np.uint64(0)), np.append(w, 0.7)
    h = _lib.vqe_hamiltonian_create(n, x, z, w)
    assert len(_lib.vqe_hamiltonian_plan(h)) >= 2
    s, l = Dev(n, dtype), Dev(n, dtype)
    try:
        g = torch.Generator(device="cuda").manual_seed(n)
        s.t.copy_(torch.complex(torch.randn(1 << n, generator=g, device="cuda", dtype=torch.float64),
                                torch.randn(1 << n, generator=g, device="cuda", dtype=torch.float64)) / 2 ** ((n + 1) / 2))
        e, _ = _lib.vqe_expect_pauli(s.h, h, _lib.EXPECT_GROUPED)
        el, _ = _lib.vqe_apply_hamiltonian(s.h, l.h, h)
        psi = s.t.to(torch.complex128)
        ref, b = torch.zeros_like(psi), torch.arange(1 << n, device="cuda")
        for xm, zm, wt in zip(x.tolist(), z.tolist(), w.tolist()):  # i^(number of Y) X^x Z^z
            q = b ^ xm
            par = q & zm
            for k in (32, 16, 8, 4, 2, 1):
                par = par ^ (par >> k)
            ref += (1 - 2 * (par & 1)).to(torch.complex128) * psi[q] * (wt * 1j ** bin(xm & zm).count("1"))
        nrm = float((psi.abs() ** 2).sum())
        E = float((psi.conj() * ref).sum().real) / nrm
        scale = np.abs(w).sum()  # bound of |H|
        assert abs(e - E) <= E_TOL[dtype] * scale and abs(el - E) <= E_TOL[dtype] * scale
        assert float((l.t.to(torch.complex128) - ref).abs().max()) <= AMP_TOL[dtype] * scale
    finally:
        s.free()
        l.free()
        _lib.vqe_hamiltonian_free(h)
