"""The coarse solve inside the two-level preconditioner: with coarse sizes that end
inside a workgroup, the preconditioner against the oracle's (tolerance 1e-3 as for
the other sizes: coarse system to 1e-6, FP32 setup and smoothing); and on both sides
of the border between vector updates inside the operator's launches and in launches
of their own (32768 coarse rows), a solve to a true residual of 1e-10."""

import numpy as np
import pytest

import fieldgen as fg
from gpuutil import from_dev, to_dev
from oracle import dirac, mg, sap
from tests.gpuutil import torch_cuda
from tests.test_gpu_default_shape import links
from tests.test_gpu_mg import DIMS, SBLK, build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 5])
def test_preconditioner_matches_oracle(n):
    U, op, lat, start, kw, P = build(n, 1)
    lat.mg_setup(to_dev(start), coarse_tol=1e-6, coarse_max_iter=2000, **kw)
    pre = mg.TwoLevel(op.D, P, mg.coarse_operator(op.D, P), sap.Blocks(DIMS, SBLK), kw["ncycles"], kw["nmr"],
                      coarse_tol=1e-12, coarse_max_iter=5000)
    r = fg.gaussian_spinor(DIMS, 63)
    x = to_dev(np.zeros_like(r))
    lat.mg_apply(to_dev(r), x)
    assert dirac.rel_l2(from_dev(x), pre(r)) <= 1e-3
    lat.close()


@pytest.mark.parametrize("n", [4, 5])  # 32768 and 40960 coarse rows
def test_solve_on_both_sides_of_the_border(n):
    from paper_2303_05883_amd import lqcd
    torch = torch_cuda()
    dims = (16, 16, 16, 16)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(361)
    field = lambda *lead: torch.view_as_complex(torch.randn((*lead, 16, 16, 16, 16, 4, 3, 2), generator=gen,
                                                            device="cuda", dtype=torch.float64))
    lat = lqcd.Lattice(dims, -1)
    lat.set_gauge(links(torch, dims, gen))
    lat.set_clover(0.11, 1.0)
    lat.mg_setup(field(n), agg=(2, 2, 2, 2), nvec=n, setup_iters=1, sap_block=(4, 4, 4, 4), ncycles=1, nmr=3)
    assert lat.mg_coarse_size() == 8192 * n
    b = field()
    x = torch.zeros_like(b)
    lat.solve_mg(b, x, tol=1e-10)
    res = b - lat.apply("D", 0, x, torch.empty_like(x))
    assert (torch.linalg.vector_norm(res) / torch.linalg.vector_norm(b)).item() <= 1e-10
    lat.close()
