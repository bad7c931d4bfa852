"""Traces of few photons where the launch rules change: the most majorants that
a small workgroup stages in LDS by itself and more, photon numbers at which the
workgroups and the queue's grabs change.  Bit for bit the tallies of one fixed
launch shape with the majorants read from memory."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2208_05247_amd import rt3d as r  # noqa: E402
from paper_2208_05247_amd import synthetic as syn  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 16, 16), (12, 19, 9), (32, 16, 16)])  # 2048, 2052 and 8192 majorants
@pytest.mark.parametrize("photons", [1, 1 << 14, (1 << 14) + 1, (1 << 15) + 1, (1 << 16) + 5, (1 << 17) - 1, 1 << 17])
def test_launch_rules(shape, photons):
    grid = syn.Grid(*shape, 50.0, 40.0, 30.0)
    df = r.DeviceFields.from_host(syn.random_fields(grid, seed=4, k_max=0.02, albedo_range=(0.1, 0.4)))
    kw = dict(brick=(1, 1, 1), diffuse_fraction=0.3)
    fixed = dict(grid_blocks=3, pool_photons=256, refill_lanes=64)
    want = r.trace(df, 50.0, 75.0, photons, 9, lds_majorant=-1, **fixed, **kw)
    got = [r.trace(df, 50.0, 75.0, photons, 9, lds_majorant=lds, **kw) for lds in (0, 1, -1)]
    med = syn.batched_cumulus(seed=2, nx=16, ny=24, nz=16, n_gp=3, photons=8, n_blobs=2).medium
    dm = r.DeviceBatchedMedium.from_host(med)
    counts = np.array([photons, 0, photons // 2 + 1], dtype=np.uint64)
    want_b, got_b = r.trace_batched(dm, 50.0, 75.0, counts, 9, **fixed), r.trace_batched(dm, 50.0, 75.0, counts, 9)
    torch.cuda.synchronize()
    for k in r.TALLY3 + r.TALLY2 + ("ledger", "stats"):
        assert all(torch.equal(want[k], g[k]) for g in got), k
        assert torch.equal(want_b[k], got_b[k]), k
