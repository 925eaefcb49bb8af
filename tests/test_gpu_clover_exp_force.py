"""Force of the exponential clover term with a lane per Hermitian block (d_R <= 3):
lattices of 16 and 24 sites, which fill a block of 32 sites partly, on Haar links
with a large c_sw, whose exponents need several squarings.  Each of s squarings
doubles the relative error of its factors, NB products' roundings each:
50 NB 2^s eps, s = 4, is 1.1e-12 for NB = 6."""
import pytest
import torch

from gpu_common import APBC, Setup, rel, wdirac
from oracle import clover_force as CF
from oracle import lattice as L
from oracle import reps as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('csw', [0.0, 0.4, 4.0])
@pytest.mark.parametrize('dims', [(2, 2, 2, 2), (2, 6, 2, 2)])
@pytest.mark.parametrize('N,rep', [(2, 'FUND'), (3, 'FUND'), (3, '2AS'), (2, 'SYM')])
def test_exp_force(N, rep, dims, csw):
    wdirac()
    m = -0.1
    s = Setup(N, rep, dims, seed=81, links='haar', precs=(0,))
    x_e = s.half(s.spinor(82), 0)[0]
    clov = s.lat.new_clover(0)
    s.lat.clover_field(clov, s.Ug, m, csw, 1, 0)
    xg = s.to_gpu_half(L.from_half(x_e, dims, 0)[None], 0)
    P = torch.zeros(dims + (4, N, N), dtype=torch.complex128, device='cuda')
    s.lat.force_eo_clover(P, xg, s.URg[0], s.Ug, clov, m, csw, 1)
    s.lat.force_clover_logdet(P, s.Ug, clov, m, csw, 1, accumulate=1)
    g = (CF.pseudofermion_force_components(x_e, s.U, rep, m, csw, APBC, dims, True)
         + CF.det_force_components(s.U, rep, m, csw, dims, True))
    assert rel(P.cpu().numpy(), R.algebra_to_matrix(g, N)) < 1.1e-12
