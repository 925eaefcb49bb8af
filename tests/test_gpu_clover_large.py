"""Clover field of a lattice just past 2^28 sites, where the site offsets of the
link and F scratch no longer fit 32 bits of bytes (SU(2) FUND with FP32 blocks, the
only call of its kind whose 283 GB fit the card).  The links are 1 but for eight
sites among the last 32, so the blocks there, and at the other ends of the rows,
equal those of a short lattice with the same links, to the bit."""
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu


def _blocks(lat, U, put):
    from paper_2503_06721_amd import wdirac as W
    U.zero_()
    U[..., 0, 0] = 1
    U[..., 1, 1] = 1
    Z = lat.dims[3]
    U[1, 1, 1, Z - 16:Z - 8] = put
    c = lat.new_clover(W.F32)
    lat.clover_field(c, U, 0.1, 1.0, 0, W.F32)
    # [parity][chirality][entry][site]: the sites of each (t, x, y) row at its last 32 and first 16 z
    rows = c.view(torch.complex64).view(2, 2, 10, -1)[..., :lat.Vh].view(2, 2, 10, 8, Z // 2)
    return rows[..., -16:].clone(), rows[..., :8].clone()


def test_past_32bit_offsets():
    from paper_2503_06721_amd import synth
    from paper_2503_06721_amd import wdirac as W
    put = torch.from_numpy(synth.haar_links((2, 2, 2, 2), 2, 3)).reshape(-1, 4, 2, 2)[:8].cuda()
    small = W.Lattice(2, 'FUND', (2, 2, 2, 64), (1, 1, 1, 1))
    exp = _blocks(small, torch.empty((2, 2, 2, 64, 4, 2, 2), dtype=torch.complex128, device='cuda'), put)
    Z = (1 << 25) + 4
    lat = W.Lattice(2, 'FUND', (2, 2, 2, Z), (1, 1, 1, 1))
    assert lat.V == (1 << 28) + 32
    need = lat.V * 4 * 4 * 16 + lat.workspace_bytes(W.OP_CLOVER) + lat.field_bytes(W.FIELD_CLOVER, 1, W.F32)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip(f'{need / 1e9:.0f} GB of device memory are not free')
    try:
        got = _blocks(lat, torch.empty((2, 2, 2, Z, 4, 2, 2), dtype=torch.complex128, device='cuda'), put)
        assert (exp[0] - exp[1][..., :1]).abs().max() > 0.01
        for e, g in zip(exp, got):
            assert torch.equal(e, g)
    finally:
        torch.cuda.empty_cache()
