"""What a trace prepares in its workspace: the majorants and level maxima that
the packing kernels form in a wave (rows of a power of two of cells) and in
launches of their own (other rows), for rows of 1 cell to more than a wave,
cell counts that end inside a wave, zeros, negative zeros and cloud-free
levels; and what a trace clears in its outputs.  All values are maxima of the
inputs, so equality is exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2208_05247_amd import rt3d as r  # noqa: E402
from paper_2208_05247_amd import synthetic as syn  # noqa: E402

pytestmark = pytest.mark.gpu


def align(n):
    return (n + 255) // 256 * 256


def section(ws, at, n):
    return ws[at:at + 4 * n].clone().view(torch.float32).cpu().numpy()


BRICKS = [((8, 8, 8), (1, 1, 1)), ((12, 6, 4), (2, 3, 2)), ((12, 10, 6), (4, 5, 3)), ((40, 9, 5), (8, 3, 5)),
          ((64, 3, 2), (16, 1, 2)), ((96, 2, 3), (32, 2, 3)), ((64, 5, 3), (64, 5, 1)), ((256, 2, 2), (128, 1, 1)),
          ((15, 4, 4), (3, 2, 4)), ((35, 3, 3), (5, 1, 1))]


def cloud_of(grid, seed):
    k = np.random.default_rng(seed).uniform(0.001, 0.02, (grid.nz, grid.ny, grid.nx)).astype(np.float32)
    k[k < 0.006] = 0.0
    k[0, 0, 0] = -0.0
    k[grid.nz // 2] = 0.0
    return k


@pytest.mark.parametrize("shape,brick", BRICKS)
def test_majorants(shape, brick):
    grid = syn.Grid(*shape, 50.0, 40.0, 30.0)
    f = syn.random_fields(grid, seed=5, k_max=0.02, albedo_range=(0.1, 0.4))
    df = r.DeviceFields.from_host(f)
    df.k_ext.copy_(torch.from_numpy(np.maximum(cloud_of(grid, 1), 0.0)))
    df.k_ext_cloud.copy_(df.k_ext)
    ws = r.alloc_workspace(int(r.workspace_size(grid, r.options(brick=brick)))).fill_(255)
    out = r.trace(df, 30.0, 10.0, 500, 3, brick=brick, workspace=ws)
    nmaj = shape[0] * shape[1] * shape[2] // (brick[0] * brick[1] * brick[2])
    want = r.majorant_build(grid, df.k_ext, brick).cpu().numpy().ravel()
    assert np.array_equal(section(ws, 512, nmaj), want)
    # the same photons on top: twice everything, nothing cleared
    twice = {k: v.clone() for k, v in out.items() if isinstance(v, torch.Tensor)}
    r.trace(df, 30.0, 10.0, 500, 3, brick=brick, workspace=ws, out=twice, accumulate=True)
    for k in r.TALLY3 + r.TALLY2 + ("ledger", "stats"):
        assert torch.equal(twice[k], 2 * out[k]), k
    # and over what is there: all of it cleared
    again = {k: torch.full_like(v, 77) for k, v in twice.items() if isinstance(v, torch.Tensor)}
    r.trace(df, 30.0, 10.0, 500, 3, brick=brick, workspace=ws, out=again)
    for k in r.TALLY3 + r.TALLY2 + ("ledger", "stats"):
        assert torch.equal(again[k], out[k]), k


@pytest.mark.parametrize("shape,brick", BRICKS)
def test_factored_majorants(shape, brick):
    grid = syn.Grid(*shape, 50.0, 40.0, 30.0)
    rng = np.random.default_rng(2)
    ngp = 3
    k_gas = rng.uniform(1e-5, 1e-4, (ngp, grid.nz)).astype(np.float32)
    cloud = cloud_of(grid, 4)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    dm = r.DeviceBatchedMedium(grid, up(k_gas), up(np.full((ngp, grid.nz), 0.5)), up(cloud),
                               up(np.full(cloud.shape, 0.99)), up(np.full(cloud.shape, 0.85)),
                               up(np.full((grid.ny, grid.nx), 0.2)))
    ws = r.alloc_workspace(int(r.workspace_size_batched(grid, ngp, r.options(brick=brick)))).fill_(255)
    r.trace_batched(dm, 30.0, 10.0, [40, 0, 25], 3, brick=brick, workspace=ws)
    bx, by, bz = brick
    mx, my, mz = shape[0] // bx, shape[1] // by, shape[2] // bz
    level = np.maximum(cloud, 0.0).reshape(grid.nz, my, by, mx, bx).max(axis=(2, 4))
    want = (k_gas[:, :, None, None] + level[None]).reshape(ngp, mz, bz, my, mx).max(axis=2)
    clear = level.reshape(mz, bz, my, mx).max(axis=1) == 0.0
    want = np.where(clear[None], -want, want)
    at = 256 + align(8 * (3 * ngp + 2))
    assert np.array_equal(section(ws, at, want.size), want.ravel())
    first = ws[256:256 + 8 * (2 * ngp + 2)].clone().view(torch.int64).cpu().numpy()
    passes, rest = np.array([40, 0, 25]) // (shape[0] * shape[1]), np.array([40, 0, 25]) % (shape[0] * shape[1])
    assert np.array_equal(first[:ngp + 1], np.concatenate([[0], np.cumsum(passes)]))
    assert np.array_equal(first[ngp + 1:], np.concatenate([[0], np.cumsum(rest)]))
