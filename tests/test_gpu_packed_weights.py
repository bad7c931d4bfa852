"""Convolutions with packed weights: bitwise the same call without a workspace
(the products and their order are the same), the data gradient bitwise the
flipped weights' convolution; one and two channel slabs, odd counts of 32
outputs, two inputs, upsampling, ragged tiles."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def call(name, *args):
    from paper_2208_05247_amd import denoise as dn
    conv = [dn._p(a) if a is None or isinstance(a, torch.Tensor) else ctypes.byref(a) if isinstance(a, dn._Conv) else a
            for a in args]
    return getattr(dn.load(), name)(*conv, dn._s())


@pytest.mark.parametrize("D,H,W,c1,c2,cout,up", [
    (2, 8, 32, 64, 0, 64, 0), (3, 9, 33, 16, 32, 96, 0), (1, 1, 1, 16, 0, 32, 0), (4, 18, 34, 128, 64, 32, 1),
    (6, 10, 2, 32, 16, 128, 1)])
def test_packed_weights_bitwise(D, H, W, c1, c2, cout, up):
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(cout + W)
    rnd = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16).cuda()
    cin = c1 + c2
    x1, x2 = rnd(D >> up, H >> up, W >> up, c1), rnd(D, H, W, c2) if c2 else None
    w, b = rnd(cout, 27, cin), torch.randn(cout, generator=g).cuda()
    c = dn._Conv(D, H, W, c1, c2, cout, 3, up, 0)
    n = 2 * cout * 27 * cin
    out = lambda ch, f=torch.bfloat16: torch.full((D, H, W, ch), 7.0, dtype=f, device="cuda")
    ref, got, short = out(cout), out(cout), out(cout)
    assert call("rt3d_dn_conv3d_fwd", c, x1, x2, w, b, 1, ref, None, cout, None) == 0
    work = torch.empty(n, dtype=torch.uint8, device="cuda")
    assert call("rt3d_dn_conv3d_fwd_ws", c, x1, x2, w, b, 1, got, None, cout, None, work, n) == 0
    assert call("rt3d_dn_conv3d_fwd_ws", c, x1, x2, w, b, 1, short, None, cout, None, work, n - 1) == 0  # not used
    assert torch.equal(ref, got) and torch.equal(ref, short)
    if cout == 32:
        hw, hb = rnd(32, 32), torch.randn(32, generator=g).cuda()
        hr, hg = out(2, torch.float32), out(2, torch.float32)
        assert call("rt3d_dn_conv3d_fwd_head", c, x1, x2, w, b, 1, hw, hb, 2, hr) == 0
        assert call("rt3d_dn_conv3d_fwd_head_ws", c, x1, x2, w, b, 1, hw, hb, 2, hg, work, n) == 0
        assert torch.equal(hr, hg)
    if cin % 32 == 0 and not up:
        dz = rnd(D, H, W, cout)
        wt = torch.empty(cin, 27, cout, dtype=torch.bfloat16, device="cuda")
        dn.flip(w, cout, cin, 3, wt)
        ref, got = out(cin), out(cin)
        dn.conv_fwd(dz, None, wt, None, False, cin, 3, y1=ref)
        dn.conv_dgrad(dz, w, cin, got)
        assert torch.equal(ref, got)
        grad = dn._Conv(D, H, W, cout, 0, cin, 3, 0, 0)
        assert call("rt3d_dn_conv3d_dgrad", grad, dz, w, got, None, cin, None, 0) == 1  # RT3D_EINVAL: no workspace
