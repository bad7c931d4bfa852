"""The single-g-point tracer with a deposit buffer behind its workspace, and
its launch rule for few photons: tallies bit for bit those of the plain
workspace in one launch shape, at the edges of the buffer's chunks, tiles and
bins and of the queue's grabs.  All sums are of integers, so equality is
exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2208_05247_amd import rt3d as r  # noqa: E402
from paper_2208_05247_amd import synthetic as syn  # noqa: E402

pytestmark = pytest.mark.gpu

KEYS = r.TALLY3 + r.TALLY2 + ("ledger", "stats")


def fields(grid, seed, k_max=0.02):
    return r.DeviceFields.from_host(syn.random_fields(grid, seed=seed, k_max=k_max, albedo_range=(0.1, 0.4)))


def workspace(grid, brick, spare):
    """The needed workspace and exactly `spare` bytes more."""
    n = int(r.workspace_size(grid, r.options(brick=brick)))
    ws = r.alloc_workspace(n + spare)
    assert ws.numel() == n + spare
    return ws


def same(a, b):
    torch.cuda.synchronize()
    for k in KEYS:
        assert torch.equal(a[k], b[k]), k
    led = [int(v) for v in r.as_uint64(a["ledger"])]
    assert led[0] + led[5] == sum(led[1:5]) + led[6] + led[7]


# cells: one bin exactly (2^13), one cell row more, several bins with a ragged
# last one, LDS majorants left out; buffers of the smallest size taken (256
# tiles and the lanes' state), one tile more, one round's worth
@pytest.mark.parametrize("shape,brick,lds", [((32, 16, 16), (8, 8, 8), 0), ((32, 16, 17), (4, 4, 1), 0),
                                             ((40, 33, 25), (5, 3, 5), 0), ((40, 33, 25), (5, 3, 5), -1)])
@pytest.mark.parametrize("spare", [90 << 20, (90 << 20) + 140000, 1 << 30])
def test_buffer_equals_atomics(shape, brick, lds, spare):
    grid = syn.Grid(*shape, 50.0, 40.0, 30.0)
    df = fields(grid, 3)
    kw = dict(brick=brick, diffuse_fraction=0.2, lds_majorant=lds)
    print("buffer case", shape, brick, lds, spare, flush=True)
    photons = (1 << 24) + 12345
    ref = r.trace(df, 35.0, 20.0, photons, 7, workspace=workspace(grid, brick, 0), **kw)
    got = r.trace(df, 35.0, 20.0, photons, 7, workspace=workspace(grid, brick, spare), **kw)
    same(got, ref)
    # added to what is there; one atomic per deposit in both
    r.trace(df, 35.0, 20.0, photons, 8, workspace=workspace(grid, brick, 0), out=ref, accumulate=True, merge=False, **kw)
    r.trace(df, 35.0, 20.0, photons, 8, workspace=workspace(grid, brick, spare), out=got, accumulate=True, merge=False,
            **kw)
    same(got, ref)


def test_photons_capped_across_rounds():
    """Photons stopped by max_iters, strong absorption (sums beyond 32 bits)
    and a buffer that fills several times."""
    grid = syn.Grid(24, 24, 24, 50.0, 50.0, 50.0)
    f = syn.uniform_fields(grid, 0.02, 0.01, 0.3, 0.5, 0.3)
    df = r.DeviceFields.from_host(f)
    kw = dict(brick=(4, 4, 4), max_iters=9, rr_threshold=0.05)
    a = r.trace(df, 10.0, 0.0, 1 << 25, 5, workspace=workspace(grid, (4, 4, 4), 0), **kw)
    b = r.trace(df, 10.0, 0.0, 1 << 25, 5, workspace=workspace(grid, (4, 4, 4), 90 << 20), **kw)
    same(b, a)
    assert int(a["stats"][r.STATS.index("capped")]) > 0


@pytest.mark.parametrize("photons", [1, 15, 16, 17, 63, 64, 65, 1025, 4096 * 16 + 1, 300000])
def test_few_photons_any_launch_shape(photons):
    """The automatic launch (small workgroups and queue grabs) against one
    workgroup with full grabs."""
    grid = syn.Grid(18, 15, 20, 50.0, 40.0, 30.0)
    df = fields(grid, 4)
    kw = dict(brick=(3, 5, 4), diffuse_fraction=0.3, photon_offset=11)
    a = r.trace(df, 50.0, 75.0, photons, 9, **kw)
    b = r.trace(df, 50.0, 75.0, photons, 9, grid_blocks=1, pool_photons=256, refill_lanes=64, **kw)
    same(a, b)
    assert int(a["stats"][0]) == photons
    med = syn.batched_cumulus(seed=2, nx=16, ny=24, nz=16, n_gp=3, photons=8, n_blobs=2).medium
    dm = r.DeviceBatchedMedium.from_host(med)
    counts = np.array([photons, 0, photons // 2 + 1], dtype=np.uint64)
    a = r.trace_batched(dm, 50.0, 75.0, counts, 9)
    b = r.trace_batched(dm, 50.0, 75.0, counts, 9, grid_blocks=1, pool_photons=256, refill_lanes=64)
    same(a, b)
