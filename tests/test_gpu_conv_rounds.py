"""The 3x3x3 convolution's tiles of three rows a wave, taken where they waste
less of the last round of workgroups: grids cut in x, y and z, one and two
channel slabs, two inputs, upsampling.  Whole-number inputs, so every FP32 sum
is exact (below 2^24) and the results have to be equal; the grids beside them
take four rows."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,W,c1,c2,cout,up", [
    (32, 260, 32, 16, 0, 64, 0), (31, 260, 33, 16, 0, 64, 0), (32, 259, 31, 16, 32, 64, 0), (32, 130, 32, 16, 0, 128, 0),
    (32, 260, 32, 32, 16, 64, 1), (32, 256, 32, 16, 0, 64, 0)])
def test_three_row_tiles(D, H, W, c1, c2, cout, up):
    from paper_2208_05247_amd import denoise as dn
    from test_gpu_conv_tiles import reference
    g = torch.Generator().manual_seed(H + W + cout)
    ints = lambda *s: torch.randint(-3, 4, s, generator=g).float().cuda()
    x1, x2 = ints(D >> up, H >> up, W >> up, c1), ints(D, H, W, c2) if c2 else None
    w, b = ints(cout, 27, c1 + c2), ints(cout)
    full = x1 if not up else x1.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)
    ref = reference(torch.cat([full, x2], 3) if c2 else full, w, b)
    lo = lambda t: None if t is None else t.to(torch.bfloat16)
    yf = torch.full((D, H, W, cout), 7.0, device="cuda")
    dn.conv_fwd(lo(x1), lo(x2), lo(w), b, False, cout, 3, yf=yf, up1=bool(up))
    assert torch.equal(yf, ref)
    y = dn.bf16_empty(D, H, W, cout)
    dn.conv_fwd(lo(x1), lo(x2), lo(w), b, True, cout, 3, y1=y, up1=bool(up))
    assert torch.equal(y, ref.clamp(min=0).to(torch.bfloat16))
