"""The 3x3x3 convolution in each of its tile sizes (4, 2 and 1 rows a wave, 2
and 1 planes; 64 and 32 output channels; with and without packed weights), on
grids that cut the tiles.  Whole-number inputs: every FP32 sum is exact (below
2^24), so the results have to be equal.  The head in one launch against the two
launches, bitwise."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def reference(x, w, b):
    D, H, W, _ = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    y = b.repeat(D * H * W, 1)
    for t in range(27):
        y += xp[t // 9:t // 9 + D, (t // 3) % 3:(t // 3) % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[3]) @ w[:, t].t()
    return y.view(D, H, W, -1)


@pytest.mark.parametrize("D,H,W,c1,c2,cout,up", [
    (33, 121, 65, 16, 0, 64, 0), (33, 121, 65, 16, 32, 64, 0), (17, 41, 33, 16, 0, 64, 0), (17, 41, 33, 32, 16, 128, 0),
    (17, 19, 33, 16, 0, 64, 0), (18, 20, 34, 16, 48, 64, 1), (5, 7, 33, 16, 16, 64, 0), (1, 1, 1, 32, 32, 64, 0),
    (33, 241, 65, 16, 0, 32, 0), (17, 81, 33, 16, 32, 32, 0), (17, 37, 33, 16, 0, 32, 0), (3, 5, 31, 48, 0, 32, 0),
    (18, 42, 34, 16, 32, 96, 1)])
def test_conv_tiles(D, H, W, c1, c2, cout, up):
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(D * 100 + H + cout)
    ints = lambda *s: torch.randint(-3, 4, s, generator=g).float().cuda()
    x1, x2 = ints(D >> up, H >> up, W >> up, c1), ints(D, H, W, c2) if c2 else None
    w, b = ints(cout, 27, c1 + c2), ints(cout)
    full = x1 if not up else x1.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)
    ref = reference(torch.cat([full, x2], 3) if c2 else full, w, b)
    lo = lambda t: None if t is None else t.to(torch.bfloat16)
    args = (lo(x1), lo(x2), lo(w), b)
    yf = torch.full((D, H, W, cout), 7.0, device="cuda")
    dn.conv_fwd(*args, False, cout, 3, yf=yf, up1=bool(up))
    assert torch.equal(yf, ref)
    y = dn.bf16_empty(D, H, W, cout)
    dn.conv_fwd(*args, True, cout, 3, y1=y, up1=bool(up))
    assert torch.equal(y, ref.clamp(min=0).to(torch.bfloat16))
    if cout == 32:
        hw, hb = lo(ints(32, 32)), ints(32)
        two, one = (torch.full((D, H, W, n), 7.0, device="cuda") for n in (2, 2))
        dn.conv_fwd(y, None, hw, hb, False, 32, 1, yf=two, yf_cols=2)
        dn.conv_fwd_head(*args, True, hw, hb, one, up1=bool(up))
        assert torch.equal(two, one)
