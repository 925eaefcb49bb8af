"""The hop's launch shape of a context with no option set, against the
colour-split form with one hop per phase (variant 1, one rhs per block) on the
same packed fields: every representation, precision and number of right-hand
sides the rule tells apart, on lattices smaller than a tile, with a ragged last
tile and (for the sub-lattice sweep) with rows of whole tiles.

Both forms add the same 8 d_R products per output element in the same order;
the compact form's link entries may differ by a few roundings each.  With
|U| entries at most 1 and d_R <= 15 the accumulated difference is below 8 d_R
+ 8 units of rounding of the largest partial sum, which the Gaussian inputs
bound by 16 d_R^(1/2): the tolerance is 64 d_R^(3/2) eps of the largest output.
"""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

BC = (-1, 1, -1, 1)
REPS = [(2, 'FUND'), (3, 'FUND'), (4, 'FUND'), (2, 'ADJ'), (3, 'ADJ'), (4, 'ADJ'), (2, 'SYM'), (3, 'SYM'), (4, 'SYM'),
        (3, '2AS'), (4, '2AS')]


def _links(dims, N, seed):
    from paper_2503_06721_amd import synth
    return torch.from_numpy(synth.haar_links(dims, N, seed)).cuda()


def _compare(N, rep, dims, prec, nrhs):
    from paper_2503_06721_amd import wdirac as W
    lat, ref = W.Lattice(N, rep, dims, BC), W.Lattice(N, rep, dims, BC)
    for opt, v in ((W.OPT_HOP_VARIANT_F64, 1), (W.OPT_HOP_VARIANT_F32, 1), (W.OPT_HOP_NR_F64, 1),
                   (W.OPT_HOP_NR_F32, 1)):
        ref.set_option(opt, v)
    UR = lat.new_links(prec)
    lat.rep_links(UR, _links(dims, N, 7), prec)
    g = torch.Generator(device='cuda').manual_seed(11)
    dt = lat.spinor_dtype(prec)
    full = torch.randn((nrhs,) + dims + (4, lat.d), dtype=dt, device='cuda', generator=g)
    xfull = torch.randn((nrhs,) + dims + (4, lat.d), dtype=dt, device='cuda', generator=g)
    eps = torch.finfo(torch.float64 if prec == W.F64 else torch.float32).eps
    for parity, dagger in ((0, 0), (1, 1)):
        inp, add = lat.pack_half(full, 1 - parity, nrhs, prec), lat.pack_half(xfull, parity, nrhs, prec)
        for kw in ({}, dict(alpha=0.7, x_add=add, beta=-1.3)):
            out = []
            for lt in (lat, ref):
                o = lt.new_half(nrhs, prec)
                lt.dslash_eo(o, inp, UR, parity, dagger=dagger, nrhs=nrhs, prec=prec, **kw)
                out.append(lt.unpack_half(o, parity, nrhs, prec))
            scale = out[1].abs().max()
            assert scale > 0
            assert (out[0] - out[1]).abs().max() <= 64 * lat.d ** 1.5 * eps * scale, (parity, dagger, kw.keys())


@pytest.mark.parametrize('prec', [0, 1])
@pytest.mark.parametrize('N,rep', REPS)
def test_small_and_ragged(N, rep, prec):
    for dims in ((2, 2, 2, 2), (4, 6, 2, 10)):
        for nrhs in (1, 2, 3, 4, 5, 6, 12):
            _compare(N, rep, dims, prec, nrhs)


@pytest.mark.parametrize('prec', [0, 1])
@pytest.mark.parametrize('N,rep', [(3, 'SYM'), (4, '2AS')])
@pytest.mark.parametrize('dims', [(2, 6, 8, 24), (4, 8, 16, 32), (2, 2, 8, 16), (16, 16, 16, 8)])
def test_sweeps_and_thresholds(N, rep, prec, dims):
    """Rows of 3, 8, 2 and 2 tiles of 32 sites; the last lattice has 16384 half-lattice sites."""
    for nrhs in (1, 2, 4, 12):
        _compare(N, rep, dims, prec, nrhs)


@pytest.mark.parametrize('N,rep,nrhs', [(2, 'ADJ', 3), (2, 'FUND', 1), (2, 'ADJ', 1)])
def test_large(N, rep, nrhs):
    """65536 half-lattice sites (three rhs per block) and 262144 (no XCD ranges)."""
    from paper_2503_06721_amd import wdirac as W
    _compare(N, rep, (32, 16, 16, 16) if nrhs > 1 else (32, 32, 32, 16), W.F64, nrhs)
