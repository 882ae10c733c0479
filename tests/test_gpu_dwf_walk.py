"""The domain-wall kernels' walk over regions and bricks on lattices whose
extents leave odd regions, bricks of one site and partly filled workgroups:
every site is computed once and from its own neighbours."""

import numpy as np
import pytest

import fieldgen as fg
from oracle import dirac, dwf
from tests.gpuutil import TOL, from_dev, lattice, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 1), ((2, 6, 2, 4), 7), ((6, 10, 14, 4), 5), ((12, 2, 6, 10), 3),
                                     ((16, 4, 4, 6), 12), ((32, 6, 4, 2), 2), ((4, 4, 2, 2), 130)])
def test_walk_covers_every_site(dims, Ls):
    U = fg.gauge_field(dims, 311, "smooth", 0.3)
    rng = np.random.default_rng(312)
    shape = (Ls,) + dims[::-1] + (4, 3)
    psi = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    op = dwf.DomainWall(U, 1.8, 0.05, Ls, -1, 1.5, 0.5)
    lat = lattice(dims, U, 0.12, 0.0)
    want = {False: op.D(psi), True: op.Ddag(psi)}
    for prec in (0, 1):
        for dag in (False, True):
            out = to_dev(np.zeros_like(psi))
            lat.dwf_apply(Ls, 1.8, 0.05, prec, to_dev(psi), out, dag=dag, b5=1.5, c5=0.5)
            assert dirac.rel_l2(from_dev(out), want[dag]) <= TOL[prec], (prec, dag)
    lat.close()
