"""Staggered CG on both sides of the border between partial sums added by the next
update and by kernels of their own (1536 workgroups of 256 sites per parity), and
with a last workgroup that is not full: a solve that runs out of iterations leaves
the x of that many steps, and a full one reaches the tolerance on the full operator."""

import pytest

from tests.gpuutil import torch_cuda
from tests.test_gpu_default_shape import links

pytestmark = pytest.mark.gpu

MASS = 0.3


@pytest.mark.parametrize("dims", [(10, 6, 6, 6), (32, 32, 32, 24), (32, 32, 30, 26)])  # 1080, 393216 | 399360 sites
def test_staggered_cg(dims):
    from paper_2303_05883_amd import lqcd
    torch = torch_cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(381)
    lat = lqcd.Lattice(dims, -1)
    lat.set_gauge(links(torch, dims, gen))
    lx, ly, lz, lt = dims
    b = torch.view_as_complex(torch.randn((lt, lz, ly, lx, 3, 2), generator=gen, device="cuda", dtype=torch.float64))
    norm = lambda v: torch.linalg.vector_norm(v).item()
    D = lambda v: lat.stag_apply("D", 0, MASS, v, torch.empty_like(v))
    hop = lambda v: D(v) - MASS * v
    t, z, y, x = torch.meshgrid(*[torch.arange(n, device="cuda") for n in (lt, lz, ly, lx)], indexing="ij")
    even = ((t + z + y + x) % 2 == 0)[..., None]
    # 6 steps on (m^2 - H_eo H_oe) x_e = m b_e - H_eo b_o from zero, x_o rebuilt
    r = even * (MASS * b - hop(b))
    xs, p, rr = torch.zeros_like(b), r.clone(), norm(r) ** 2
    for _ in range(6):
        q = even * (MASS ** 2 * p - hop(hop(p)))
        alpha = rr / torch.sum(p.conj() * q).real
        xs, r = xs + alpha * p, r - alpha * q
        rn = norm(r) ** 2
        p, rr = r + rn / rr * p, rn
    want = xs + ~even * (b - hop(xs)) / MASS
    got = torch.zeros_like(b)
    st = lat.stag_solve(MASS, b, got, max_iter=6, raise_on_fail=False)
    assert st.status == lqcd.ENOCONV and st.inner_iters == 6
    assert norm(got - want) <= 1e-12 * norm(want)
    for prec in (0, 1):
        got.zero_()
        lat.stag_solve(MASS, b, got, tol=1e-11, inner_prec=prec)
        assert norm(b - D(got)) <= 1e-11 * norm(b)
    lat.close()
