"""Links at an address that is a multiple of 8 bytes but not of 16, as a caller's
slice of a larger buffer may have: the kernels that load link entries directly into
LDS take another way and give the same results."""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu


def _shifted(t):
    """A copy of t 8 bytes past a 16-byte boundary."""
    raw = t.contiguous().view(torch.uint8).reshape(-1)
    out = torch.empty(raw.numel() + 24, dtype=torch.uint8, device='cuda')
    out = out[(8 - out.data_ptr()) % 16:][:raw.numel()]
    out.copy_(raw)
    assert out.data_ptr() % 16 == 8
    return out


@pytest.mark.parametrize('N', [2, 3, 4])
def test_gauge_kernels(N):
    """The same sums in the same order: equal to the bit."""
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    dims = (2, 4, 6, 4)
    lat = W.Lattice(N, 'FUND', dims, (1, 1, 1, 1))
    U = torch.from_numpy(synth.haar_links(dims, N, 5)).cuda()
    V = _shifted(U)
    F, G = torch.zeros_like(U), torch.zeros_like(U)
    lat.gauge_force(F, U, 5.3)
    lat.gauge_force(G, V, 5.3)
    assert F.abs().max() > 0 and torch.equal(F, G)
    assert lat.gauge_action(U, 5.3) == lat.gauge_action(V, 5.3)


@pytest.mark.parametrize('N,rep', [(3, 'SYM'), (4, '2AS')])
@pytest.mark.parametrize('form', [None, 6])
def test_multi_rhs_hop(N, rep, form):
    """The colour-split form in place of the multi-rhs form: sums in another order, 48 products of order one."""
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    dims, nrhs = (4, 6, 8, 24), 12
    lat = W.Lattice(N, rep, dims)
    if form:
        lat.set_option(W.OPT_HOP_VARIANT_F64, form)
    UR = lat.new_links()
    lat.rep_links(UR, torch.from_numpy(synth.haar_links(dims, N, 7)).cuda())
    g = torch.Generator(device='cuda').manual_seed(3)
    v = lat.pack_half(torch.randn((nrhs,) + dims + (4, lat.d), dtype=torch.complex128, device='cuda', generator=g), 1,
                      nrhs)
    a, b = lat.new_half(nrhs), lat.new_half(nrhs)
    lat.dslash_eo(a, v, UR, 0, nrhs=nrhs)
    lat.dslash_eo(b, v, _shifted(UR), 0, nrhs=nrhs)
    a, b = lat.unpack_half(a, 0, nrhs), lat.unpack_half(b, 0, nrhs)
    assert (a - b).abs().max() <= 1e-13 * a.abs().max()
