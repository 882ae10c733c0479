"""The SAP block kernel on every block size it takes (64, 128, 192 and 256
sites), on blocks of extent 1 (both neighbours outside) and on long rows,
against the oracle; tolerance as in test_gpu_sap.py."""

import numpy as np
import pytest

import fieldgen as fg
from oracle import dirac, sap
from tests.gpuutil import from_dev, lattice, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block,csw", [((32, 8, 2, 2), (16, 4, 1, 1), 1.0), ((4, 8, 4, 16), (2, 4, 2, 8), 1.0),
                                            ((12, 8, 8, 4), (6, 4, 4, 2), 1.0), ((12, 8, 8, 4), (6, 4, 4, 2), 0.0),
                                            ((16, 8, 4, 4), (8, 4, 2, 1), 1.0), ((32, 4, 8, 4), (16, 2, 4, 2), 0.0),
                                            ((8, 8, 8, 8), (4, 4, 4, 4), 1.2)])
def test_block_sizes(dims, block, csw):
    kappa = 0.13
    U = fg.gauge_field(dims, 331, "smooth", 0.3)
    eta = fg.gaussian_spinor(dims, 332)
    op = dirac.Operator(U, kappa, csw)
    lat = lattice(dims, U, kappa, csw)
    want = sap.sap(op.D, sap.Blocks(dims, block), eta, 2, 3)
    got = from_dev(lat.apply_sap(to_dev(eta), to_dev(np.zeros_like(eta)), block, 2, 3))
    assert dirac.rel_l2(got, want) <= 5e-5
    lat.close()
