"""The deposit buffer at the edges of its rule: the fewest bins (128 of 8192
cells), one cell layer less (atomics in both), a ragged last bin, the fewest
photons and one less; buffers of many rounds and of few.  Tallies bit for bit
those of the plain workspace; all sums are of integers, so equality is exact."""
import pytest

torch = pytest.importorskip("torch")

from paper_2208_05247_amd import rt3d as r  # noqa: E402
from paper_2208_05247_amd import synthetic as syn  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,brick", [((128, 64, 128), (8, 8, 8)), ((128, 64, 127), (8, 8, 1)),
                                         ((110, 99, 97), (5, 3, 1)), ((100, 110, 130), (4, 5, 10))])
@pytest.mark.parametrize("photons,spare", [(1 << 22, 96 << 20), ((1 << 22) + 777, 1 << 30), ((1 << 22) - 1, 96 << 20)])
def test_buffer_rule(shape, brick, photons, spare):
    grid = syn.Grid(*shape, 50.0, 40.0, 30.0)
    df = r.DeviceFields.from_host(syn.random_fields(grid, seed=6, k_max=0.01, albedo_range=(0.1, 0.4)))
    print("bins case", shape, brick, photons, spare, flush=True)
    n = int(r.workspace_size(grid, r.options(brick=brick)))
    ref, got = (r.trace(df, 35.0, 20.0, photons, 7, brick=brick, diffuse_fraction=0.1, workspace=r.alloc_workspace(n + s))
                for s in (0, spare))
    torch.cuda.synchronize()
    for k in r.TALLY3 + r.TALLY2 + ("ledger", "stats"):
        assert torch.equal(ref[k], got[k]), k
