"""Weight and bias gradients at the edges of the 3x3x3 kernel's tiles: each
channel tiling (2 x 1, 1 x 1, 1 x 2 and 1 x 3 tiles of 32), a half-filled input
tile, inputs split inside a tile, voxel tiles cut in x and y, single planes,
more chunks than one tile has planes and fewer units than workgroups; against
FP64 sums of the same BF16 values.  FP32 accumulation of n products is within
n^0.5 2^-24 relative of them (3e-6 at the 2e3 terms here); 1e-5 is asked."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def reference(x, dz):
    D, H, W, _ = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    g = dz.reshape(-1, dz.shape[3]).t().contiguous()
    return torch.stack([g @ xp[t // 9:t // 9 + D, (t // 3) % 3:(t // 3) % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[3])
                        for t in range(27)], dim=1), g.sum(dim=1)


@pytest.mark.parametrize("D,H,W,c1,c2,cout", [
    (3, 4, 32, 32, 0, 64), (1, 5, 33, 16, 0, 32), (2, 1, 7, 16, 32, 64), (5, 9, 31, 48, 16, 32), (2, 3, 65, 64, 32, 32),
    (40, 4, 32, 32, 0, 32), (7, 6, 40, 16, 80, 32), (3, 8, 34, 32, 16, 96), (1, 1, 1, 64, 0, 128), (16, 17, 3, 96, 32, 64)])
def test_weight_gradient_edges(D, H, W, c1, c2, cout):
    from paper_2208_05247_amd import denoise as dn
    g = torch.Generator().manual_seed(D * 1000 + W)
    x = torch.randn(D, H, W, c1 + c2, generator=g).to(torch.bfloat16)
    dz = torch.randn(D, H, W, cout, generator=g).to(torch.bfloat16)
    rw, rb = reference(x.double(), dz.double())
    x1 = x[..., :c1].contiguous().cuda()
    x2 = x[..., c1:].contiguous().cuda() if c2 else None
    rel = lambda a, b: float((a.double().cpu() - b).norm() / b.norm())
    start = torch.randn(cout, 27, c1 + c2, generator=g)
    for ws in (None, torch.empty(dn.wgrad_workspace_size(x1, x2, cout, 3), dtype=torch.uint8, device="cuda")):
        dw, db = start.cuda(), torch.ones(cout, device="cuda")
        dn.conv_wgrad(x1, x2, dz.cuda(), cout, 3, dw, db, workspace=ws)
        assert rel(dw, rw + start) < 1e-5 and rel(db, rb + 1.0) < 1e-5
        only = torch.zeros_like(dw)
        dn.conv_wgrad(x1, x2, dz.cuda(), cout, 3, only, None, workspace=ws)  # no bias gradient wanted
        assert rel(only, rw) < 1e-5
