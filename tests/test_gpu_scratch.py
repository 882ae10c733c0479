"""Device blocks kept by a context between calls: every call gives the same bits
on a context that has made other calls of other sizes as on a fresh one, whatever
those left in the blocks (sources of 1e150, whose norms overflow)."""

import numpy as np
import pytest

import fieldgen as fg
from tests.gpuutil import from_dev, lattice, to_dev

pytestmark = pytest.mark.gpu

DIMS = (8, 4, 4, 8)


def calls(lat, fill=1.0):
    """Outputs of every kind of call that takes blocks from the pool."""
    from paper_2303_05883_amd import lqcd
    rng = np.random.default_rng(391)
    gauss = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    sp = to_dev(fill * gauss(*DIMS[::-1], 4, 3))
    col = to_dev(fill * gauss(*DIMS[::-1], 3))
    out = []

    def run(f, b, **kw):
        x = to_dev(np.zeros(tuple(b.shape), dtype=np.complex128))
        try:
            f(b, x, **kw)
        except lqcd.LqcdError:
            assert fill != 1.0
        out.append(from_dev(x))

    for prec in (lqcd.F64, lqcd.F32):
        run(lambda b, x: lat.stag_apply("D", prec, 0.2, b, x), col)
        run(lambda b, x: lat.stag_solve(0.2, b, x, inner_prec=prec), col)
    run(lambda b, x: lat.solve_sap(b, x, block=(4, 2, 2, 4), ncycles=2, nmr=3), sp)
    for ls in (4, 6):
        b5 = to_dev(fill * gauss(ls, *DIMS[::-1], 4, 3))
        run(lambda b, x: lat.dwf_apply(ls, 1.8, 0.05, lqcd.F64, b, x, b5=1.5, c5=0.5), b5)
        run(lambda b, x: lat.dwf_solve(ls, 1.8, 0.05, b, x, b5=1.5, c5=0.5), b5)
        for prec in (lqcd.F64, lqcd.F32):
            run(lambda b, x: lat.dwf_solve_eo(ls, 1.8, 0.05, b, x, b5=1.5, c5=0.5, inner_prec=prec), b5)
    return out


def test_kept_blocks_do_not_show():
    U = fg.gauge_field(DIMS, 392, "smooth", 0.3)
    lat = lattice(DIMS, U, 0.12, 1.0)
    want = calls(lat)
    calls(lat, 1e150)
    assert all(np.array_equal(g, w) for g, w in zip(calls(lat), want))
    fresh = lattice(DIMS, U, 0.12, 1.0)
    assert all(np.array_equal(g, w) for g, w in zip(calls(fresh), want))
    fresh.close()
    lat.close()
