"""WDIRAC_OPT_CG_CHECK_EVERY on a lattice that iterates inside one kernel: a kernel
runs the iterations of one interval and hands x, p and r on in memory, so the
interval changes no bit; and it acts, which only the time shows: a check is two
host calls and a launch, 10 us or more, beside iterations of about 10 us, a factor
of 2 over 400 of each, of which the test asks 1.2, the fastest of five each."""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu


def test_interval():
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    dims, n = (4, 4, 4, 4), 400
    lat = W.Lattice(2, 'FUND', dims)
    UR = lat.new_links()
    lat.rep_links(UR, torch.from_numpy(synth.expH_links(dims, 2, 0.3, 5)).cuda())
    g = torch.Generator(device='cuda').manual_seed(6)
    b = lat.pack_half(torch.randn((1,) + dims + (4, 2), dtype=torch.complex128, device='cuda', generator=g), 0)
    ws = lat.new_workspace(W.OP_CG)
    out, best = {}, {}
    for every in (None, 1000, 7, 1):
        if every:
            lat.set_option(W.OPT_CG_CHECK_EVERY, every)
        t = []
        for _ in range(5):
            x = lat.new_half()
            rc, st = lat.cg_eo(x, b, UR, 0.1, tol=1e-100, maxit=n, workspace=ws)
            assert rc == W.ENOCONV and st[0]['iters'] == n
            t.append(st[0]['seconds'])
        out[every], best[every] = x, min(t)
    print({k: round(v * 1e6) for k, v in best.items()}, flush=True)
    for x in out.values():
        assert torch.equal(x, out[None])
    assert best[1] > 1.2 * best[1000]
