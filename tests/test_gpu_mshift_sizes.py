"""Multi-shift CG with a smallest shift above zero, whose step length needs |p|^2:
a partial sum of it per block of the base update, which on small lattices with a
large d_R are more than the hop's tiles."""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

BC = (-1, 1, 1, 1)


def _check(N, rep, dims, shifts, m0=-0.2, tol=1e-9):
    """||b - (A + s) x_s|| <= tol ||b|| with A applied by apply_dhat; the residual formed once more in FP64 rounds
    far below the margin of 1e-3 tol."""
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    lat = W.Lattice(N, rep, dims, BC)
    UR = lat.new_links()
    lat.rep_links(UR, synth.expH_links_torch(dims, N, 0.3, 3))
    g = torch.Generator(device='cuda').manual_seed(4)
    b = lat.pack_half(torch.randn((1,) + dims + (4, lat.d), dtype=torch.complex128, device='cuda', generator=g), 0)
    x = lat.new_shift_fields(len(shifts))
    rc, st = lat.cg_mshift_eo(x, b, UR, m0, shifts, tol=tol, allow=())
    assert rc == W.OK and all(s['iters'] > 0 for s in st)
    u, q = lat.new_half(), lat.new_half()
    for k, s in enumerate(shifts):
        xk = lat.shift_field(x, k)
        lat.apply_dhat(u, xk, UR, m0)
        lat.apply_dhat(q, u, UR, m0, dagger=1)
        lat.axpby(q, 1.0, q, s, xk)
        lat.axpby(q, 1.0, b, -1.0, q)
        assert lat.norm2(q)[0] <= (1.001 * tol) ** 2 * lat.norm2(b)[0], (k, s)


@pytest.mark.parametrize('dims', [(2, 2, 2, 2), (2, 2, 4, 34), (4, 6, 8, 10)])
@pytest.mark.parametrize('N,rep', [(4, 'SYM'), (4, 'ADJ')])
def test_small_lattices(N, rep, dims):
    """1, 2 and 4 blocks a component group; d_R = 10 and 15."""
    _check(N, rep, dims, [0.02, 0.5])


@pytest.mark.parametrize('shifts', [[0.3], [0.05, 0.4, 2.0]])
def test_long_rows(shifts):
    """5120 partial sums of |r|^2, more than a block of the base update adds up itself, and 1280 blocks of it with a
    thread for all components of a site."""
    _check(2, 'ADJ', (32, 32, 32, 20), shifts)
