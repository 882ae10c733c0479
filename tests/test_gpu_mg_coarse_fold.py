"""The coarse solve on both sides of the bound on partial sums that each workgroup of
the next launch adds for itself: 196608 coarse rows (all sums so), 212992 (alpha
and omega by kernels of their own) and 425984 (beta too). The preconditioned solve
reaches a true residual of 1e-10 and two solves give the same bits."""

import pytest

from tests.gpuutil import torch_cuda
from tests.test_gpu_default_shape import links

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lz,n", [(16, 12), (16, 13), (32, 13)])
def test_solve(lz, n):
    from paper_2303_05883_amd import lqcd
    torch = torch_cuda()
    dims = (16, 16, lz, 32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(411)
    field = lambda *lead: torch.view_as_complex(torch.randn((*lead, 32, lz, 16, 16, 4, 3, 2), generator=gen,
                                                            device="cuda", dtype=torch.float64))
    lat = lqcd.Lattice(dims, -1)
    lat.set_gauge(links(torch, dims, gen))
    lat.set_clover(0.11, 1.0)
    lat.mg_setup(field(n), agg=(2, 2, 2, 2), nvec=n, setup_iters=1, sap_block=(4, 4, 4, 4), ncycles=1, nmr=3)
    assert lat.mg_coarse_size() == 16 * 16 * lz * 32 // 16 * 2 * n
    b = field()
    xs = [torch.zeros_like(b) for _ in range(2)]
    for x in xs:
        lat.solve_mg(b, x, tol=1e-10)
    res = b - lat.apply("D", 0, xs[0], torch.empty_like(b))
    assert (torch.linalg.vector_norm(res) / torch.linalg.vector_norm(b)).item() <= 1e-10
    assert torch.equal(xs[0], xs[1])
    lat.close()
