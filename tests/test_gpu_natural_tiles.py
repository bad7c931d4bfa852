"""The convolution with weights as the caller has them, around the number of
workgroups from which it takes its large tiles (129): bitwise the call with
packed weights, which takes them from 512 on (the products of an output and their
order are the same in every tile)."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_packed_weights import call  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,W,c1,c2,cout,up", [(16, 64, 64, 64, 0, 64, 0), (25, 39, 63, 64, 0, 64, 0), (25, 39, 63, 48, 0, 96, 0),
                                                 (26, 40, 64, 32, 16, 64, 1), (13, 37, 65, 64, 0, 128, 0)])
def test_tiles_of_natural_weights(D, H, W, c1, c2, cout, up):
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(D + cout)
    rnd = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16).cuda()
    x1, x2 = rnd(D >> up, H >> up, W >> up, c1), rnd(D, H, W, c2) if c2 else None
    w, b = rnd(cout, 27, c1 + c2), torch.randn(cout, generator=g).cuda()
    c = dn._Conv(D, H, W, c1, c2, cout, 3, up, 0)
    n = 2 * cout * 27 * (c1 + c2)
    got, want = (torch.full((D, H, W, cout), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    assert call("rt3d_dn_conv3d_fwd", c, x1, x2, w, b, 1, got, None, cout, None) == 0
    work = torch.empty(n, dtype=torch.uint8, device="cuda")
    assert call("rt3d_dn_conv3d_fwd_ws", c, x1, x2, w, b, 1, want, None, cout, None, work, n) == 0
    assert torch.equal(got, want)
