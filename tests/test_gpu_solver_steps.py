"""The solver's fused iteration kernels: CG on lattices below a tile, with a
ragged tile, and with more partial sums than a block adds up itself; the
multi-shift recursion with every grouping of its deferred updates."""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

BC = (-1, 1, 1, 1)


def _system(N, rep, dims, nrhs, seed=3):
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    lat = W.Lattice(N, rep, dims, BC)
    if np.prod(dims) > 1 << 16:
        U = synth.expH_links_torch(dims, N, 0.3, seed)
    else:
        U = torch.from_numpy(synth.expH_links(dims, N, 0.3, seed)).cuda()
    UR, UR32 = lat.new_links(W.F64), lat.new_links(W.F32)
    lat.rep_links(UR, U, W.F64)
    lat.rep_links(UR32, U, W.F32)
    g = torch.Generator(device='cuda').manual_seed(seed)
    b = lat.pack_half(torch.randn((nrhs,) + dims + (4, lat.d), dtype=torch.complex128, device='cuda', generator=g), 0,
                      nrhs)
    return W, lat, UR, UR32, b


@pytest.mark.parametrize('mode', [0, 1])
@pytest.mark.parametrize('N,rep,dims,nrhs', [(2, 'FUND', (2, 2, 2, 2), 1), (3, 'FUND', (4, 6, 2, 10), 3),
                                             (3, 'SYM', (4, 4, 4, 8), 4), (3, '2AS', (4, 4, 4, 8), 12),
                                             (2, 'ADJ', (32, 32, 32, 20), 1)])
def test_cg_residual(N, rep, dims, nrhs, mode):
    """||b - A x|| <= tol ||b|| with A applied by apply_dhat (the last lattice: 5120 tiles); the residual is formed
    once more in FP64, whose rounding (below 1e-13 of ||b||) is far under the margin of 1e-3 tol."""
    W, lat, UR, UR32, b = _system(N, rep, dims, nrhs)
    m0, tol = -0.2, 1e-8
    x = lat.new_half(nrhs)
    rc, st = lat.cg_eo(x, b, UR, m0, tol=tol, nrhs=nrhs, mode=mode, UR32=UR32, allow=())
    assert rc == W.OK and all(s['iters'] > 0 for s in st)
    u, q = lat.new_half(nrhs), lat.new_half(nrhs)
    lat.apply_dhat(u, x, UR, m0, nrhs=nrhs)
    lat.apply_dhat(q, u, UR, m0, dagger=1, nrhs=nrhs)
    lat.axpby(q, 1.0, b, -1.0, q, nrhs=nrhs)
    for r2, b2 in zip(lat.norm2(q, nrhs), lat.norm2(b, nrhs)):
        assert r2 <= (1.001 * tol) ** 2 * b2


@pytest.mark.parametrize('shifts', [[0.0], [0.3], [0.0, 0.05], [0.01, 3.0, 0.4, 0.07, 20.0]])
def test_mshift_grouping(shifts):
    """How many iterations run between host checks changes neither the updates nor their order: the solutions are the
    same to the bit for every interval (1: one deferred update at a time; 3, 11: groups cut by the ring)."""
    W, lat, UR, _, b = _system(3, 'FUND', (4, 6, 4, 10), 1)
    out = []
    for every in (4, 1, 3, 11):
        lat.set_option(W.OPT_CG_CHECK_EVERY, every)
        x = lat.new_shift_fields(len(shifts))
        rc, st = lat.cg_mshift_eo(x, b, UR, -0.2, shifts, tol=1e-9, allow=())
        assert rc == W.OK
        out.append([lat.unpack_half(lat.shift_field(x, k), 0) for k in range(len(shifts))])
    for o in out[1:]:
        for a, c in zip(o, out[0]):
            assert torch.equal(a, c)
    u, q = lat.new_half(), lat.new_half()
    for k, s in enumerate(shifts):
        xk = lat.pack_half(out[0][k], 0)
        lat.apply_dhat(u, xk, UR, -0.2)
        lat.apply_dhat(q, u, UR, -0.2, dagger=1)
        lat.axpby(q, 1.0, q, s, xk)
        lat.axpby(q, 1.0, b, -1.0, q)
        assert lat.norm2(q)[0] <= (1.001e-9) ** 2 * lat.norm2(b)[0]
