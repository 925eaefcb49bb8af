"""Clover blocks where the elimination has to pivot: a large c_sw on Haar links
makes the odd-site blocks indefinite, and lattices of 16 and 24 sites leave the
last group of lanes short of a matrix.  Oracle: NumPy inverse and log-determinant
of the oracle's blocks.  An inverse from partial pivoting carries an error of
order NB eps cond: the tolerance is 50 NB eps times the largest condition number
of the blocks; for log|det| of n blocks it is the same per block."""
import numpy as np
import pytest
import torch

from gpu_common import Setup, rel, wdirac
from oracle import clover as CL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('dims', [(2, 2, 2, 2), (2, 6, 2, 2)])
@pytest.mark.parametrize('N,rep', [(2, 'FUND'), (3, 'FUND'), (2, 'ADJ'), (4, 'FUND'), (3, 'SYM'), (4, '2AS')])
def test_indefinite_blocks(N, rep, dims):
    W = wdirac()
    s = Setup(N, rep, dims, seed=71, links='haar', precs=(0,))
    m, csw = -3.0, 9.0
    M = CL.diagonal_blocks(s.UR, m, csw, False)
    Mo = CL.half_blocks(M, dims, 1)
    assert np.linalg.eigvalsh(Mo).min() < 0 < np.linalg.eigvalsh(Mo).max()
    nb = Mo.shape[-1]
    tol = 50 * nb * np.finfo(float).eps * np.linalg.cond(Mo).max()
    psi = s.spinor(72)
    c = s.lat.new_clover(W.F64)
    s.lat.clover_field(c, s.Ug, m, csw, 0, W.F64)
    out = s.lat.new_half()
    s.lat.apply_clover(out, s.to_gpu_half(psi, 1, 0), c, 1)
    exp = CL.apply_sitewise(np.linalg.inv(Mo), s.half(psi, 1)[0])
    assert rel(s.from_gpu_half(out, 1, 1, 0)[0], exp) < tol
    ld = s.lat.clover_logdet(c)
    sign, ref = np.linalg.slogdet(Mo)
    assert abs(ld - ref.sum()) <= tol * ref.size
