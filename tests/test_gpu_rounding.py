"""Rounding of the operators against the same in long double: the Wilson hop and the
clover blocks stay as accurate as sums of products that are rounded first.

The bounds lie half way between the two orders emulated on the CPU (every
multiply-add in long double, rounded once). Hop, links exp(0.3 i H): products first
1.36e-16, serial multiply-adds 1.42e-16. A psi on this lattice, its blocks rounded to
FP64: 1.46e-16 and 1.80e-16 (1.00e-16 with the diagonal added last); FP32 2^29 times
that."""

import numpy as np
import pytest

import fieldgen as fg
from oracle import dirac
from tests.gpuutil import from_dev, lattice, to_dev

DIMS, KAPPA, CSW = (8, 8, 8, 8), 0.137, 1.0
LD = np.clongdouble


def fields():
    """Links, links with the third row rebuilt in long double, A in long double, a source."""
    U = fg.gauge_field(DIMS, 1003, "smooth", 0.3)
    V = U.astype(LD)
    for a in range(3):
        i, j = (a + 1) % 3, (a + 2) % 3
        V[..., 2, a] = (V[..., 0, i] * V[..., 1, j] - V[..., 0, j] * V[..., 1, i]).conj()
    A = np.zeros(DIMS[::-1] + (12, 12), LD)
    A[...] = np.eye(12)
    for mu in range(4):
        for nu in range(mu + 1, 4):
            f = dirac.field_strength(V, mu, nu)[..., None, :, None, :]
            A += np.longdouble(KAPPA) * CSW * (dirac.sigma(mu, nu)[:, None, :, None] * f).reshape(A.shape)
    return U, V, A, fg.gaussian_spinor(DIMS, 77)


def error(got, want):
    d = (from_dev(got) - want).astype(np.complex128)
    return np.linalg.norm(d) / np.linalg.norm(want.astype(np.complex128))


@pytest.mark.gpu
def test_hop_and_clover():
    import torch
    U, V, A, psi = fields()
    x = to_dev(psi)
    even, odd = dirac.mask(psi, 0), dirac.mask(psi, 1).astype(LD)
    lat = lattice(DIMS, U, KAPPA, 0.0)
    want = dirac.mask(dirac.hop(V, odd, -1), 0)
    for block, split, planes in ((64, 1, 1), (64, 2, 1), (64, 4, 1), (32, 0, 4)):
        lat.set_hop_shape(0, block, split, planes, 0)
        assert error(lat.apply("HOP_EO", 0, x, torch.empty_like(x)), want) <= 1.39e-16, split
    lat.close()
    lat = lattice(DIMS, U, KAPPA, CSW)
    want = dirac.site_apply(A, even.astype(LD))
    for prec, bound in ((0, 1.63e-16), (1, 1.63e-16 * 2 ** 29)):
        assert error(lat.apply("DEE", prec, x, torch.empty_like(x)), want) <= bound, prec
    lat.close()
