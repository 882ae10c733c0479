"""The launch shape a context starts with, at sizes on both sides of each of the
rule's borders: valid on the lattice, and the Schur operator it gives agrees with
one lane per site in site order (FP64 reference) to the precision's tolerance."""

import pytest

from tests.gpuutil import TOL, torch_cuda

pytestmark = pytest.mark.gpu

# sites per parity: 12000 | 12096, 32256 | 33280 | 40960, 119808 | 122880 | 140800, 249600 | 253440, 451584, 802816
SIZES = [(20, 20, 10, 6), (12, 12, 12, 14), (16, 16, 14, 18), (16, 16, 10, 26), (16, 16, 16, 20),
         (16, 26, 24, 24), (16, 16, 24, 40), (16, 20, 22, 40), (16, 24, 26, 50), (24, 22, 24, 40), (24, 28, 28, 48),
         (32, 28, 28, 64)]


def links(torch, dims, gen):
    """SU(3) links on the GPU: rows 0 and 1 of complex Gaussian matrices orthonormalised."""
    lx, ly, lz, lt = dims
    g = torch.randn((lt, lz, ly, lx, 4, 2, 3, 2), generator=gen, device="cuda", dtype=torch.float64)
    g = torch.view_as_complex(g)
    r0 = g[..., 0, :] / torch.linalg.vector_norm(g[..., 0, :], dim=-1, keepdim=True)
    r1 = g[..., 1, :] - (r0.conj() * g[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    r2 = torch.linalg.cross(r0, r1).conj()
    return torch.stack([r0, r1, r2], -2).contiguous()


@pytest.mark.parametrize("dims", SIZES)
def test_default_shape(dims):
    from paper_2303_05883_amd import lqcd
    torch = torch_cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(341)
    lat = lqcd.Lattice(dims, -1)
    lat.set_gauge(links(torch, dims, gen))
    lat.set_clover(0.12, 1.0)
    lx, ly, lz, lt = dims
    psi = torch.view_as_complex(torch.randn((lt, lz, ly, lx, 4, 3, 2), generator=gen, device="cuda",
                                            dtype=torch.float64))
    got = [lat.apply("DPREC_SCHUR", prec, psi, torch.empty_like(psi)) for prec in range(3)]
    for prec in range(3):
        lat.set_hop_shape(prec, *lat.get_hop_shape(prec))  # raises for a shape that does not fit
    lat.set_hop_shape(0)
    want = lat.apply("DPREC_SCHUR", 0, psi, torch.empty_like(psi))
    for prec in range(3):
        err = torch.linalg.vector_norm(got[prec] - want) / torch.linalg.vector_norm(want)
        assert err.item() <= TOL[prec], prec
    lat.close()
