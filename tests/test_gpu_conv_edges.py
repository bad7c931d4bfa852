"""The 3x3x3 convolution at the edges of its tiles: 64- and 32-channel slabs
(and both in one layer), outputs split between two tensors, single planes and
rows, rows of 31 to 33 voxels, inputs at half resolution, BF16 outputs that
are not 16-byte aligned; against FP64 (FP32 accumulation of 27 cin BF16
products: 1e-5 relative) and, between output forms, bit for bit."""
import pytest

torch = pytest.importorskip("torch")

from oracle import denoise_ref as dr  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,W,c1,c2,cout,o1,up", [
    (1, 1, 1, 16, 0, 64, 64, False), (2, 7, 31, 32, 0, 96, 32, False), (3, 8, 32, 16, 16, 128, 96, False),
    (4, 10, 34, 32, 16, 160, 64, True), (2, 16, 64, 64, 32, 32, 32, True), (5, 17, 33, 16, 32, 64, 32, False),
    (2, 2, 2, 48, 0, 32, 32, True), (1, 9, 65, 16, 0, 192, 192, False)])
def test_conv_edges(D, H, W, c1, c2, cout, o1, up):
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(D + 10 * W + cout)
    s = 2 if up else 1
    x1 = torch.randn(D // s, H // s, W // s, c1, generator=g).to(torch.bfloat16)
    x2 = torch.randn(D, H, W, c2, generator=g).to(torch.bfloat16) if c2 else None
    w = (torch.randn(cout, 27, c1 + c2, generator=g) * 0.1).to(torch.bfloat16)
    b = torch.randn(cout, generator=g)
    full = x1.double()
    if up:
        full = full.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)
    if x2 is not None:
        full = torch.cat([full, x2.double()], 3)
    ref = dr.conv(full.permute(3, 0, 1, 2).unsqueeze(0), w.double(), b.double(), 3)[0].permute(1, 2, 3, 0)
    dev = lambda t: None if t is None else t.cuda()
    args = (dev(x1), dev(x2), dev(w), dev(b))
    yf = torch.empty(D, H, W, cout, device="cuda")
    dn.conv_fwd(*args, False, cout, 3, yf=yf, up1=up)
    assert float((yf.double().cpu() - ref).norm() / ref.norm()) < 1e-5
    want = yf.to(torch.bfloat16)
    for pad in (0, 1):  # 1: outputs start 2 bytes into their storage
        y1 = torch.full((D * H * W * o1 + pad,), 7.0, dtype=torch.bfloat16, device="cuda")[pad:].view(D, H, W, o1)
        y2 = torch.full((D * H * W * (cout - o1) + pad,), 7.0, dtype=torch.bfloat16, device="cuda")[pad:]
        y2 = y2.view(D, H, W, cout - o1) if o1 < cout else None
        dn.conv_fwd(*args, False, cout, 3, y1=y1, y2=y2, o1=o1, up1=up)
        assert torch.equal(y1, want[..., :o1].contiguous())
        assert y2 is None or torch.equal(y2, want[..., o1:].contiguous())
