"""The 16-byte forms of the backward pass's elementwise kernels against the
one-element forms (which run where a tensor is not 16-byte aligned), and the
fused steps against the separate calls: bit for bit, the roundings are the
same."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def bits(t):
    return t.contiguous().view(torch.int16)


def make(g, shape, shift):
    """BF16 values, signs and zeros among them; shift 1: 2 bytes into their storage."""
    n = 1
    for v in shape:
        n *= v
    v = torch.randn(n, generator=g).to(torch.bfloat16).cuda()
    v[::7] = 0
    t = torch.empty(n + shift, dtype=torch.bfloat16, device="cuda")[shift:]
    t.copy_(v)
    return t.view(shape)


@pytest.mark.parametrize("D,H,W,C", [(2, 2, 2, 8), (1, 1, 1, 32), (3, 5, 7, 24), (4, 2, 6, 64), (2, 3, 33, 40)])
def test_wide_forms_equal_narrow(D, H, W, C):
    from paper_2208_05247_amd import denoise as dn
    res = []
    for shift in (0, 1):
        g = torch.Generator().manual_seed(C)
        small, big = make(g, (D, H, W, C), shift), make(g, (2 * D, 2 * H, 2 * W, C), shift)
        other, act = make(g, big.shape, shift), make(g, big.shape, shift)
        actc = make(g, small.shape, shift)
        new = lambda like: make(g, like.shape, shift)
        out = {}
        out["up2"] = dn.up2(small, out=new(big))
        out["up2_bwd"] = dn.up2(big, backward=True, out=new(small))
        out["pool2_bwd"] = dn.pool2(small, backward=True, out=new(big))
        for name, f in (("relu_bwd", dn.relu_bwd), ("add", dn.add)):
            o = new(big)
            f(big, act, o)
            out[name] = o
        if shift == 0:
            o = new(small)
            dn.relu_bwd(out["up2_bwd"], actc, o)
            assert torch.equal(bits(dn.up2_relu_bwd(big, actc, new(small))), bits(o))
            o, de = new(big), other.clone()
            dn.add(other, out["pool2_bwd"], o)
            dn.relu_bwd(o, act, o)
            assert torch.equal(bits(dn.pool2_add_relu_bwd(small, de, act, de)), bits(o))  # in place
        res.append(out)
    for k in res[0]:
        assert torch.equal(bits(res[0][k]), bits(res[1][k])), k


@pytest.mark.parametrize("cpad,nout", [(8, 2), (32, 2), (32, 9), (16, 16)])
def test_loss_rows(cpad, nout):
    """The loss kernel by rows against the residual head written out."""
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(cpad + nout)
    nvox = 1003
    out = torch.randn(nvox, cpad, generator=g).cuda()
    base, target = torch.randn(nvox, nout, generator=g).cuda(), torch.randn(nvox, nout, generator=g).cuda()
    pred = torch.empty_like(base)
    dout = torch.full((nvox, cpad), 7.0, dtype=torch.bfloat16, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    dn._check(dn.load().rt3d_dn_mse(dn._p(out), cpad, dn._p(base), dn._p(target), nout, nvox, dn._p(pred), dn._p(dout),
                                    dn._p(loss), dn._s()), "mse")
    want = out[:, :nout] + base
    assert torch.equal(pred, want)
    d = want - target
    grad = torch.zeros(nvox, cpad, device="cuda")
    grad[:, :nout] = d * torch.tensor(2.0 / (nvox * nout), dtype=torch.float64).float().item()
    assert torch.equal(bits(dout), bits(grad.to(torch.bfloat16)))
    assert abs(loss.item() - (d.double() ** 2).sum().item()) <= 1e-12 * loss.item()
