"""The launch rule of the hop on both sides of its lines on size and number of
right-hand sides, against the colour-split form with one hop per phase (as
test_gpu_default_shape.py, whose tolerance it takes)."""
import pytest

from test_gpu_default_shape import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('N,rep,dims,prec,nrhs', [
    # SU(4) SYM FP64: 256 blocks of one rhs, and more
    (4, 'SYM', (8, 8, 8, 8), 0, 8), (4, 'SYM', (8, 8, 8, 8), 0, 10),
    # SU(3) SYM FP64 without a sweep: 711 and 790 compact blocks; too large
    (3, 'SYM', (10, 10, 10, 10), 0, 9), (3, 'SYM', (10, 10, 10, 10), 0, 10), (3, 'SYM', (10, 14, 6, 18), 0, 12),
    (3, 'SYM', (18, 14, 14, 14), 0, 8),
    # d_R = 6 FP32: groups of two against three and four
    (4, '2AS', (12, 12, 12, 12), 1, 6), (4, '2AS', (16, 8, 12, 16), 1, 6), (3, 'SYM', (10, 10, 10, 10), 1, 8),
    (3, 'SYM', (10, 14, 6, 18), 1, 8), (3, 'SYM', (8, 8, 8, 6), 1, 12),
    # SU(2) SYM with one rhs per block, d_R = 4 with two
    (2, 'SYM', (10, 10, 10, 10), 0, 7), (2, 'SYM', (10, 14, 8, 18), 0, 5), (4, 'FUND', (18, 14, 14, 14), 0, 2),
    (4, 'FUND', (16, 16, 16, 8), 0, 6), (4, 'FUND', (20, 14, 14, 14), 0, 6)])
def test_lines(N, rep, dims, prec, nrhs):
    _compare(N, rep, dims, prec, nrhs)


@pytest.mark.parametrize('prec', [0, 1])
def test_xcd_ranges(prec):
    """327680 half-lattice sites: XCD ranges 640 KiB (FP64) and 320 KiB long."""
    _compare(2, 'FUND', (20, 32, 32, 32), prec, 1)
