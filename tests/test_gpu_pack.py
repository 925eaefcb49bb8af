"""Packing of half spinors through LDS: lattices below a 64-site tile, with a
remainder and filled exactly, the smallest and largest d_R, several right-hand
sides, against indexing on the host; copies, so equal to the bit."""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('prec', [0, 1])
@pytest.mark.parametrize('N,rep,dims,nrhs', [(2, 'FUND', (2, 2, 2, 2), 1), (2, 'FUND', (4, 2, 6, 4), 3),
                                             (3, 'SYM', (4, 4, 2, 4), 2), (4, 'ADJ', (2, 4, 6, 2), 5)])
def test_pack_round_trip(N, rep, dims, nrhs, prec):
    from paper_2503_06721_amd import wdirac as W
    lat = W.Lattice(N, rep, dims, (-1, 1, 1, 1))
    dt = torch.complex128 if prec == 0 else torch.complex64
    g = torch.Generator(device='cuda').manual_seed(4)
    v = torch.randn((nrhs,) + dims + (4, lat.d), dtype=torch.complex128, device='cuda', generator=g).to(dt)
    site_parity = torch.from_numpy(np.indices(dims).sum(0) % 2).cuda()
    for parity in (0, 1):
        half = lat.pack_half(v, parity, nrhs, prec)
        # packed [rhs][spin][colour][stride], sites of the parity in lexicographic order
        n = int(np.prod(dims)) // 2
        rows = half.view(dt).reshape(nrhs, 4, lat.d, -1)[..., :n]
        sites = v[:, site_parity == parity]   # [rhs][site][spin][colour]
        assert torch.equal(rows, sites.permute(0, 2, 3, 1))
        back = lat.unpack_half(half, parity, nrhs, prec).reshape(v.shape)
        assert torch.equal(back[:, site_parity == parity], sites)
