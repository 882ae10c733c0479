"""The full operator D, both parities in one launch, at sizes on both sides of the
borders of its launch rule (lanes per site, XCD slabs or site order, partial last
blocks): FP64 against the sum of its four parity blocks, each a launch of its own,
to the rounding of the order of the hops; FP32 and FP16 against FP64."""

import pytest

from tests.gpuutil import TOL, torch_cuda
from tests.test_gpu_default_shape import links

pytestmark = pytest.mark.gpu

# sites per parity: 16, 12000 | 12096, 99840 | 101376, 105600, 114400
SIZES = [(2, 2, 2, 4), (20, 20, 10, 6), (12, 12, 12, 14), (16, 24, 20, 26), (16, 24, 24, 22), (20, 24, 20, 22),
         (22, 26, 20, 20)]


@pytest.mark.parametrize("csw", [0.0, 1.0])
@pytest.mark.parametrize("dims", SIZES)
def test_full_operator(dims, csw):
    from paper_2303_05883_amd import lqcd
    torch = torch_cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(351)
    lat = lqcd.Lattice(dims, -1)
    lat.set_gauge(links(torch, dims, gen))
    lat.set_clover(0.12, csw)
    lx, ly, lz, lt = dims
    psi = torch.view_as_complex(torch.randn((lt, lz, ly, lx, 4, 3, 2), generator=gen, device="cuda",
                                            dtype=torch.float64))
    want = sum(lat.apply(n, 0, psi, torch.empty_like(psi)) for n in ("DEE", "DEO", "DOE", "DOO"))
    got = lat.apply("D", 0, psi, torch.empty_like(psi))
    # at most 8 hops of 6 products and a clover row of 6, added in another order
    assert (got - want).abs().max().item() <= 1e-14 * want.abs().max().item()
    for prec in (1, 2):
        low = lat.apply("D", prec, psi, torch.empty_like(psi))
        err = torch.linalg.vector_norm(low - got) / torch.linalg.vector_norm(got)
        assert err.item() <= TOL[prec], prec
    assert torch.equal(lat.apply("D", 0, psi, psi), got)  # in place
    lat.close()
