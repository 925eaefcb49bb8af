"""CG with the clover block in the hop's epilogue (one right-hand side): the leading
blocks of the step length, the residual update and its sums, per lattice of a batch,
in FP64 and in the FP32 inner iterations of a mixed solve.  A = D-hat^+ D-hat is
put together from dslash_eo and apply_clover; the residual formed from it rounds
far below the margin of 1e-3 tol."""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu

BC = (-1, 1, 1, 1)


@pytest.mark.parametrize('mode', [0, 1])
@pytest.mark.parametrize('N,rep,shapes', [(3, 'FUND', [(4, 6, 2, 10)]), (2, 'FUND', [(4, 4, 8, 8)]),
                                          (4, 'FUND', [(2, 4, 6, 6), (4, 4, 4, 4)]),
                                          (3, 'FUND', [(4, 4, 2, 6), (2, 2, 2, 2), (4, 6, 4, 10)])])
def test_cg_residual(N, rep, shapes, mode):
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    batch = len(shapes) > 1
    lat = W.Lattice(N, rep, shapes if batch else shapes[0], BC)
    U = torch.cat([torch.from_numpy(synth.expH_links(s, N, 0.3, 7 + k).reshape(-1, 4, N, N))
                   for k, s in enumerate(shapes)]).cuda()
    lead = (sum(int(np.prod(s)) for s in shapes),) if batch else shapes[0]
    U = U.reshape(lead + (4, N, N))
    UR, clov = {}, {}
    for prec in (0, 1):
        UR[prec], clov[prec] = lat.new_links(prec), lat.new_clover(prec)
        lat.rep_links(UR[prec], U, prec)
        lat.clover_field(clov[prec], U, -0.2, 1.3, 0, prec)
    g = torch.Generator(device='cuda').manual_seed(8)
    b = lat.pack_half(torch.randn(lead + (4, lat.d), dtype=torch.complex128, device='cuda', generator=g), 0)
    x, tol = lat.new_half(), 1e-9
    rc, st = lat.cg_eo_clover(x, b, UR[0], clov[0], tol=tol, mode=mode, UR32=UR[1], clov32=clov[1], allow=())
    assert rc == W.OK and len(st) == len(shapes) and all(s['iters'] > 5 for s in st)
    if mode:   # reliable updates, not restarts of an FP32 iteration that gains nothing
        y = lat.new_half()
        ref = lat.cg_eo_clover(y, b, UR[0], clov[0], tol=tol, allow=())[1]
        assert all(s['iters'] <= 1.5 * r['iters'] for s, r in zip(st, ref))

    def dhat(v, dagger):
        t, e, out = lat.new_half(), lat.new_half(), lat.new_half()
        lat.dslash_eo(t, v, UR[0], 1, dagger)
        lat.apply_clover(t, t, clov[0], 1)
        lat.apply_clover(e, v, clov[0], 0)
        lat.dslash_eo(out, t, UR[0], 0, dagger, alpha=1.0, x_add=e, beta=-1.0)
        return out

    q = dhat(dhat(x, 0), 1)
    lat.axpby(q, 1.0, b, -1.0, q)
    for s, r2, b2 in zip(st, lat.norm2(q), lat.norm2(b)):
        assert r2 <= (1.001 * tol) ** 2 * b2
        assert abs((r2 / b2) ** 0.5 - s['true_rel_resid']) <= 1e-3 * tol
