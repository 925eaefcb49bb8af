"""CG on lattices that iterate inside one workgroup: every colour count, the
largest lattices it takes, a single site pair per wavefront and thread counts
that fill no wavefront, against the recurrence written with operator calls."""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

BC = (-1, 1, 1, 1)


@pytest.mark.parametrize('mode', [0, 1])
@pytest.mark.parametrize('N,rep,dims,nrhs', [(2, 'FUND', (2, 2, 2, 2), 1), (2, 'FUND', (4, 4, 4, 8), 2),
                                             (3, 'FUND', (4, 4, 4, 4), 1), (3, '2AS', (4, 2, 6, 6), 3),
                                             (2, 'ADJ', (2, 6, 4, 6), 1), (4, 'FUND', (4, 4, 4, 4), 5),
                                             (2, 'FUND', (4, 4, 4, 10), 1)])
def test_iterates(N, rep, dims, nrhs, mode):
    """x after six iterations (the last lattice has more sites than one workgroup takes).  Rounding enters at eps a
    step (1e-16; 6e-8 for the FP32 inner solve) and grows by the few steps and the condition number, below 1e3."""
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    lat = W.Lattice(N, rep, dims, BC)
    U = torch.from_numpy(synth.expH_links(dims, N, 0.3, 5)).cuda()
    UR, UR32 = lat.new_links(W.F64), lat.new_links(W.F32)
    lat.rep_links(UR, U, W.F64)
    lat.rep_links(UR32, U, W.F32)
    g = torch.Generator(device='cuda').manual_seed(6)
    b = lat.pack_half(torch.randn((nrhs,) + dims + (4, lat.d), dtype=torch.complex128, device='cuda', generator=g), 0,
                      nrhs)
    m0, n = 0.1, 6
    x = lat.new_half(nrhs)
    rc, st = lat.cg_eo(x, b, UR, m0, tol=1e-13, maxit=n, nrhs=nrhs, mode=mode, UR32=UR32)
    assert rc == W.ENOCONV and [s['iters'] for s in st] == [n] * nrhs

    def apply(v):
        p, u, q = lat.pack_half(v, 0, nrhs), lat.new_half(nrhs), lat.new_half(nrhs)
        lat.apply_dhat(u, p, UR, m0, nrhs=nrhs)
        lat.apply_dhat(q, u, UR, m0, dagger=1, nrhs=nrhs)
        return lat.unpack_half(q, 0, nrhs)

    def dot(a, c):
        return (a.conj() * c).real.flatten(1).sum(1).reshape((nrhs,) + (1,) * (a.dim() - 1))

    r = lat.unpack_half(b, 0, nrhs)
    r = r.reshape((nrhs, -1))
    y, p = torch.zeros_like(r), r.clone()
    for _ in range(n):
        q = apply(p.reshape((nrhs,) + dims + (4, lat.d))).reshape(nrhs, -1)
        rho = dot(r, r)
        a = rho / dot(p, q)
        y, r = y + a * p, r - a * q
        p = r + dot(r, r) / rho * p
    got = lat.unpack_half(x, 0, nrhs).reshape(nrhs, -1)
    err = ((got - y).flatten(1).norm(dim=1) / y.flatten(1).norm(dim=1)).max().item()
    assert err < (1e-12 if mode == 0 else 1e-4)
