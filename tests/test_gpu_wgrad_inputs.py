"""The 3x3x3 weight gradient of inputs that its 16-byte loads do not take:
tensors 2 and 8 bytes into their storage, one at a time and together.  Against
FP64 sums of the same BF16 values, within the 1e-5 of the aligned call (FP32
accumulation of n products: n^0.5 2^-24 relative, 3e-6 at the 2e3 terms here)."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_wgrad import reference  # noqa: E402

pytestmark = pytest.mark.gpu


def at_offset(t, elements):
    """The same values, `elements` elements into a 16-byte aligned storage."""
    s = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    v = s[elements:elements + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == 2 * elements
    return v


@pytest.mark.parametrize("c1,c2,cout,k", [(32, 0, 64, 3), (16, 32, 32, 3), (64, 32, 32, 3), (32, 0, 32, 1)])
@pytest.mark.parametrize("o1,o2,oz", [(1, 0, 0), (0, 4, 0), (0, 0, 1), (4, 1, 4)])
def test_any_alignment(c1, c2, cout, k, o1, o2, oz):
    from paper_2208_05247_amd import denoise as dn
    D, H, W = 5, 7, 35
    g = torch.Generator().manual_seed(c1 + 10 * o1 + oz)
    x = torch.randn(D, H, W, c1 + c2, generator=g).to(torch.bfloat16)
    dz = torch.randn(D, H, W, cout, generator=g).to(torch.bfloat16)
    rw, rb = reference(x.double(), dz.double())
    if k == 1:
        rw = rw[:, 13:14]
    x1, dzg = at_offset(x[..., :c1].contiguous(), o1), at_offset(dz, oz)
    x2 = at_offset(x[..., c1:].contiguous(), o2) if c2 else None
    rel = lambda a, b: float((a.double().cpu() - b).norm() / b.norm())
    for ws in (None, torch.empty(dn.wgrad_workspace_size(x1, x2, cout, k), dtype=torch.uint8, device="cuda")):
        print("alignment case", c1, c2, cout, k, o1, o2, oz, ws is not None, flush=True)
        dw, db = torch.zeros(cout, k ** 3, c1 + c2, device="cuda"), torch.zeros(cout, device="cuda")
        dn.conv_wgrad(x1, x2, dzg, cout, k, dw, db, workspace=ws)
        assert rel(dw, rw) < 1e-5 and rel(db, rb) < 1e-5
        only = torch.zeros_like(dw)
        dn.conv_wgrad(x1, x2, dzg, cout, k, only, None, workspace=ws)
        assert rel(only, rw) < 1e-5


@pytest.mark.parametrize("D,H,W", [(2, 3, 33), (3, 5, 7), (1, 6, 40), (2, 7, 56), (2, 1, 47), (2, 4, 32), (1, 3, 64)])
@pytest.mark.parametrize("c1,c2,cout", [(16, 0, 32), (32, 0, 64), (48, 16, 32), (64, 32, 32)])
@pytest.mark.parametrize("what", ["input", "gradient"])
def test_infinities_at_the_domain_edge(D, H, W, c1, c2, cout, what):
    """An infinity or NaN in the last column, row or plane reaches the taps that
    meet it inside the domain and no other."""
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(W * 10 + c1)
    x = torch.randn(D, H, W, c1 + c2, generator=g).to(torch.bfloat16)
    dz = torch.randn(D, H, W, cout, generator=g).to(torch.bfloat16)
    t = x if what == "input" else dz
    t[0, 0, W - 1, 3] = float("inf")
    t[D - 1, H - 1, 0, 9] = float("-inf")
    t[D - 1, H - 1, W - 1, 12] = float("nan")
    rw, rb = reference(x.double(), dz.double())
    x1 = x[..., :c1].contiguous().cuda()
    x2 = x[..., c1:].contiguous().cuda() if c2 else None
    ws = torch.empty(dn.wgrad_workspace_size(x1, x2, cout, 3), dtype=torch.uint8, device="cuda")
    dw, db = torch.zeros(cout, 27, c1 + c2, device="cuda"), torch.zeros(cout, device="cuda")
    dn.conv_wgrad(x1, x2, dz.cuda(), cout, 3, dw, db, workspace=ws)
    for got, want in ((dw.double().cpu(), rw), (db.double().cpu(), rb)):
        ok = torch.isfinite(want)
        assert torch.equal(torch.isfinite(got), ok)
        assert float((got[ok] - want[ok]).norm()) <= 1e-5 * float(want[ok].norm())


@pytest.mark.parametrize("D,H,W,c1,c2,cout", [(1, 1, 1, 128, 0, 256), (1, 4, 32, 32, 0, 64), (3, 4, 32, 128, 0, 256),
                                              (5, 4, 32, 16, 0, 32), (16, 4, 32, 32, 0, 32), (17, 4, 32, 32, 0, 32)])
def test_few_partial_sums(D, H, W, c1, c2, cout):
    """Fewer partial sums than lane groups to add them (1, 3, 5, 16, 17 chunks)."""
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(D)
    x = torch.randn(D, H, W, c1, generator=g).to(torch.bfloat16)
    dz = torch.randn(D, H, W, cout, generator=g).to(torch.bfloat16)
    rw, rb = reference(x.double(), dz.double())
    start = torch.randn(cout, 27, c1, generator=g)
    ws = torch.empty(dn.wgrad_workspace_size(x, None, cout, 3), dtype=torch.uint8, device="cuda")
    dw, db = start.cuda(), torch.ones(cout, device="cuda")
    dn.conv_wgrad(x.cuda(), None, dz.cuda(), cout, 3, dw, db, workspace=ws)
    rel = lambda a, b: float((a.double().cpu() - b).norm() / b.norm())
    assert rel(dw, rw + start) < 1e-5 and rel(db, rb + 1.0) < 1e-5


@pytest.mark.parametrize("D,H,W,c1,c2,cout,workspace", [
    (16, 16, 24, 16, 0, 32, True), (5, 1229, 1, 16, 0, 32, True), (2, 8, 16, 256, 128, 128, True), (1, 1, 257, 256, 128, 128, True),
    (32, 32, 48, 64, 32, 32, False), (1, 127, 259, 64, 32, 32, False), (5, 13, 21, 256, 128, 128, False),
    (1, 2, 683, 256, 128, 128, False)])
def test_few_voxels(D, H, W, c1, c2, cout, workspace):
    """The most voxels that the element kernel takes for a number of channel
    tiles, with and without a workspace, and one or a few more."""
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(D + W)
    x = torch.randn(D, H, W, c1 + c2, generator=g).to(torch.bfloat16)
    dz = torch.randn(D, H, W, cout, generator=g).to(torch.bfloat16)
    rw, rb = reference(x.double(), dz.double())
    x1 = x[..., :c1].contiguous().cuda()
    x2 = x[..., c1:].contiguous().cuda() if c2 else None
    ws = torch.empty(dn.wgrad_workspace_size(x1, x2, cout, 3), dtype=torch.uint8, device="cuda") if workspace else None
    rel = lambda a, b: float((a.double().cpu() - b).norm() / b.norm())
    dw, db = torch.zeros(cout, 27, c1 + c2, device="cuda"), torch.zeros(cout, device="cuda")
    dn.conv_wgrad(x1, x2, dz.cuda(), cout, 3, dw, db, workspace=ws)
    assert rel(dw, rw) < 1e-5 and rel(db, rb) < 1e-5
