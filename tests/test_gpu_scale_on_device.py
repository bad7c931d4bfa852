"""Inference with the field scale read on the device: bitwise the calls that
take its value, over scales from 1e-30 to 1e30 (1/s is formed there in FP64 and
rounded, which is the correctly rounded FP32 quotient), and refused where the
scale is zero in FP32."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1e-30, 3.1e-9, 0.7, 12345.6, 1e30])
@pytest.mark.parametrize("cpad", [4, 8])
def test_scale_on_device(size, cpad):
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(int(cpad + abs(size) % 97))
    rnd = lambda: torch.rand(8, 16, 24, generator=g).cuda()
    hd, hf, ke, ka = rnd() * size, rnd() * size, rnd() * 0.02, rnd() * 1e-4
    extra = rnd() * size if cpad == 8 else None
    s = dn.field_scale(hd, hf)
    n, scale = hd.numel(), dn._field_scale(hd, hf)
    feat = [dn.bf16_empty(8, 16, 24, cpad) for _ in range(2)]
    base = [torch.empty(8, 16, 24, 2, device="cuda") for _ in range(2)]
    args = [dn._p(t) for t in (hd, hf, ke, ka)]
    dn._check(dn.load().rt3d_dn_features(*args, 20.0, s, n, cpad, dn._p(extra), dn._p(feat[0]), dn._p(base[0]), dn._s()), "")
    dn._check(dn.load().rt3d_dn_features_at(*args, 20.0, dn._p(scale), n, cpad, dn._p(extra), dn._p(feat[1]),
                                            dn._p(base[1]), dn._s()), "")
    assert torch.equal(feat[0].view(torch.int16), feat[1].view(torch.int16)) and torch.equal(base[0], base[1])
    out = torch.randn(8, 16, 24, 2, generator=g).cuda()
    res = [torch.empty_like(hd) for _ in range(4)]
    dn._check(dn.load().rt3d_dn_residual_unfeature(dn._p(out), 2, args[0], args[1], s, n, dn._p(res[0]), dn._p(res[1]),
                                                   dn._s()), "")
    dn._check(dn.load().rt3d_dn_residual_unfeature_at(dn._p(out), 2, args[0], args[1], dn._p(scale), n, dn._p(res[2]),
                                                      dn._p(res[3]), dn._s()), "")
    assert torch.equal(res[0], res[2]) and torch.equal(res[1], res[3])


def test_zero_scale_refused():
    from paper_2208_05247_amd import denoise as dn, rt3d
    net = dn.Denoiser(base=32, seed=1)
    h = torch.zeros(8, 8, 8, device="cuda")
    k = torch.full_like(h, 0.01)
    od, of = dn.denoise(net, h, h.clone(), k, k, 20.0)  # no heating at all: scale one
    assert bool(torch.isfinite(od).all()) and bool(torch.isfinite(of).all())
    h[0, 0, 0] = 1e-45
    with pytest.raises(rt3d.Rt3dError):
        dn.denoise(net, h, h.clone(), k, k, 20.0)


@pytest.mark.parametrize("D,H,W", [(2, 2, 2), (4, 18, 34), (2, 16, 66)])
def test_first_layer_weight_rows(D, H, W):
    """The packed first layer from the 16-channel weights: bitwise from their
    first four channels (the others, here not zero, are not used)."""
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(W)
    rnd = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16).cuda()
    x, w, b = rnd(D, H, W, 4), rnd(32, 27, 16), torch.randn(32, generator=g).cuda()
    got = []
    for weights in (w[:, :, :4].contiguous(), w):
        y, p = dn.bf16_empty(D, H, W, 32), dn.bf16_empty(D // 2, H // 2, W // 2, 32)
        dn.conv_fwd_pool(x, weights, b, True, y, p)
        got.append((y, p))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
