"""Gauge force, plaquette action and kinetic term on lattices whose sites fill a
64-site block partly, exactly and with a remainder, against the oracle: FP64
sums of a few hundred products per link, so 1e-12 relative is ample (the tests
of the trajectories use the same)."""
import numpy as np
import pytest
import torch

from gpu_common import rel, wdirac
from oracle import hmc as OH
from paper_2503_06721_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('dims', [(2, 2, 2, 2), (2, 4, 2, 4), (6, 2, 4, 2), (4, 2, 6, 6)])
@pytest.mark.parametrize('N', [2, 3, 4])
def test_gauge_kernels(N, dims):
    W = wdirac()
    lat = W.Lattice(N, 'FUND', dims, (1, 1, 1, 1))
    U = synth.haar_links(dims, N, 5)
    Ug = torch.from_numpy(U).cuda()
    beta = 5.3
    F = torch.zeros_like(Ug)
    lat.gauge_force(F, Ug, beta)
    exp = OH.gauge_force(U, beta)
    assert rel(F.cpu().numpy(), exp) < 1e-12
    lat.gauge_force(F, Ug, beta, scale=-0.25, accumulate=1)
    assert rel(F.cpu().numpy(), 0.75 * exp) < 1e-12
    assert abs(lat.gauge_action(Ug, beta) / OH.gauge_action(U, beta) - 1) < 1e-12
    g = torch.Generator(device='cuda').manual_seed(4)
    pi = torch.randn(Ug.shape, dtype=torch.complex128, device='cuda', generator=g)
    assert abs(lat.kinetic(pi) / float(pi.abs().square().sum()) - 1) < 1e-12
