"""The CG solvers keep their scalars on the GPU and enqueue iterations in
chunks: the iteration cap holds to the iteration inside a chunk, at its end and
in the next one, and the iterate at the cap is the one of that many steps."""

import numpy as np
import pytest

import fieldgen as fg
from oracle import dirac, staggered
from paper_2303_05883_amd import lqcd
from tests.gpuutil import from_dev, lattice, to_dev

pytestmark = pytest.mark.gpu

DIMS, MASS = (4, 6, 4, 8), 0.1


def oracle_cg(U, b, n):
    """n CG steps on (m^2 - H_eo H_oe) x_e = m b_e - H_eo b_o from zero, x_o rebuilt."""
    even = (dirac.parity_field(DIMS) == 0)[..., None]
    hop = lambda v: staggered.hop(U, v, -1)
    A = lambda v: even * (MASS ** 2 * v - hop(hop(v)))
    r = even * (MASS * b - hop(b))
    x, p, rr = np.zeros_like(b), r.copy(), np.vdot(r, r).real
    for _ in range(n):
        q = A(p)
        alpha = rr / np.vdot(p, q).real
        x, r = x + alpha * p, r - alpha * q
        rn = np.vdot(r, r).real
        p, rr = r + rn / rr * p, rn
    return x + ~even * (b - hop(x)) / MASS


@pytest.mark.parametrize("cap", [1, 3, 4, 5, 9])
def test_iteration_cap(cap):
    U = fg.gauge_field(DIMS, 321, "smooth", 0.3)
    rng = np.random.default_rng(322)
    b = rng.standard_normal(DIMS[::-1] + (3,)) + 1j * rng.standard_normal(DIMS[::-1] + (3,))
    lat = lattice(DIMS, U, 0.12, 0.0)
    x = to_dev(np.zeros_like(b))
    st = lat.stag_solve(MASS, to_dev(b), x, max_iter=cap, raise_on_fail=False)
    assert st.status == lqcd.ENOCONV and st.inner_iters == cap
    assert dirac.rel_l2(from_dev(x), oracle_cg(U, b, cap)) <= 1e-12
    b5 = rng.standard_normal((4,) + DIMS[::-1] + (4, 3)) + 0j
    for prec in (lqcd.F64, lqcd.F32):
        st = lat.dwf_solve_eo(4, 1.8, 0.05, to_dev(b5), to_dev(np.zeros_like(b5)), b5=1.5, c5=0.5, max_iter=cap,
                              inner_prec=prec, raise_on_fail=False)
        assert st.status == lqcd.ENOCONV and st.inner_iters == cap
    for c5 in (0.0, 0.5):
        st = lat.dwf_solve(4, 1.8, 0.05, to_dev(b5), to_dev(np.zeros_like(b5)), b5=1.5, c5=c5, max_iter=cap,
                           raise_on_fail=False)
        assert st.status == lqcd.ENOCONV and st.inner_iters == cap
    lat.close()
