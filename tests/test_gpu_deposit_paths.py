"""Traces through the deposit buffer on grids that it is used for (128 bins and
more): every option, the fewest tiles, few workgroups with tile counts one past
a multiple of the 64 tiles that the addition takes at a time, calls that
overlap, a graph.  Tallies bit for bit those of the plain workspace; all sums are
of integers, so equality is exact.  Each case checks that the buffer was taken:
the surplus of its workspace has been written."""
import pytest

torch = pytest.importorskip("torch")

from paper_2208_05247_amd import rt3d as r  # noqa: E402
from paper_2208_05247_amd import synthetic as syn  # noqa: E402
from test_deposit_plan_cpu import spare_for  # noqa: E402

pytestmark = pytest.mark.gpu

KEYS = r.TALLY3 + r.TALLY2 + ("ledger", "stats")
LANES = 768  # of a workgroup


def fields(shape, seed=6, k_max=0.01):
    grid = syn.Grid(*shape, 50.0, 40.0, 30.0)
    return r.DeviceFields.from_host(syn.random_fields(grid, seed=seed, k_max=k_max, albedo_range=(0.1, 0.4)))


def plain(df, brick):
    """The needed workspace and nothing more."""
    return r.alloc_workspace(int(r.workspace_size(df.grid, r.options(brick=brick))))


def buffered(df, brick, spare):
    """The needed workspace and `spare` bytes, which hold a pattern."""
    n = int(r.workspace_size(df.grid, r.options(brick=brick)))
    ws = r.alloc_workspace(n + spare)
    ws[n:] = 0x5a
    return ws


def used(df, brick, ws):
    n = int(r.workspace_size(df.grid, r.options(brick=brick)))
    return bool((ws[n:n + 16384 * 8] != 0x5a).any())


def same(a, b):
    torch.cuda.synchronize()
    for k in KEYS:
        assert torch.equal(a[k], b[k]), k
    led = [int(v) for v in r.as_uint64(a["ledger"])]
    assert led[0] + led[5] == sum(led[1:5]) + led[6] + led[7]


@pytest.mark.parametrize("shape,brick", [((128, 64, 128), (8, 8, 8)), ((104, 100, 104), (8, 4, 8))])
@pytest.mark.parametrize("groups,tiles", [(7, 1025), (32, 1089)])
def test_few_workgroups(shape, brick, groups, tiles):
    df = fields(shape)
    photons = (1 << 22) + 5
    spare = spare_for(df.grid, r.options(brick=brick), photons, groups * LANES, tiles)
    print("deposit case", shape, brick, groups, tiles, spare, flush=True)
    kw = dict(brick=brick, diffuse_fraction=0.1, grid_blocks=groups)
    ws = buffered(df, brick, spare)
    got = r.trace(df, 35.0, 20.0, photons, 7, workspace=ws, **kw)
    ref = r.trace(df, 35.0, 20.0, photons, 7, workspace=plain(df, brick), **kw)
    same(got, ref)
    assert used(df, brick, ws)


def zeroed(df):
    t = r.alloc_tallies(df.grid)
    for v in t.values():
        v.zero_()
    return t


def test_calls_that_overlap_add_to_the_same_tallies():
    """Two calls over disjoint photons that accumulate on two streams, each with
    a buffer of its own: no deposit of either is lost."""
    df, brick, n = fields((128, 64, 128)), (8, 8, 8), 1 << 23
    kw = dict(brick=brick, diffuse_fraction=0.1, accumulate=True)
    ref = r.trace(df, 35.0, 20.0, 2 * n, 7, workspace=plain(df, brick), out=zeroed(df), **kw)
    spaces = [buffered(df, brick, 192 << 20) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    out = zeroed(df)
    torch.cuda.synchronize()
    for k in range(2):
        print("overlap case", k, flush=True)
        r.trace(df, 35.0, 20.0, n, 7, photon_offset=k * n, workspace=spaces[k], out=out, stream=streams[k], **kw)
    torch.cuda.synchronize()
    for k in r.TALLY3 + r.TALLY2 + ("stats",):
        assert torch.equal(out[k], ref[k]), k
    for k in ("incoming", "toa", "sfc", "rr_gain", "rr_loss", "lost"):
        assert out["ledger"][r.LEDGER.index(k)] == ref["ledger"][r.LEDGER.index(k)], k
    assert all(used(df, brick, ws) for ws in spaces)


def test_ledger_of_a_short_call_within_a_long_one():
    """The ledger's heating entries are the sums of the tallies once all calls
    have ended, also where one began and ended while another ran."""
    df, brick = fields((64, 64, 64)), (8, 8, 8)
    kw = dict(brick=brick, accumulate=True)
    out = zeroed(df)
    r.trace(df, 35.0, 20.0, 1 << 14, 3, workspace=plain(df, brick), out=out, **kw)
    spaces, streams = [plain(df, brick) for _ in range(2)], [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    r.trace(df, 35.0, 20.0, 1 << 26, 7, workspace=spaces[0], out=out, stream=streams[0], **kw)
    r.trace(df, 35.0, 20.0, 1 << 12, 8, workspace=spaces[1], out=out, stream=streams[1], **kw)
    torch.cuda.synchronize()
    led = [int(v) for v in r.as_uint64(out["ledger"])]
    assert led[2] == int(out["abs_dir"].sum()) and led[3] == int(out["abs_dif"].sum())
    assert led[0] + led[5] == sum(led[1:5]) + led[6] + led[7]


def test_one_array_for_direct_and_diffuse_heating():
    """Both heating tallies in one array: their sum."""
    df, brick, n = fields((128, 64, 128)), (8, 8, 8), 1 << 22
    kw = dict(brick=brick, diffuse_fraction=0.3)
    ref = r.trace(df, 35.0, 20.0, n, 7, workspace=plain(df, brick), **kw)
    out = r.alloc_tallies(df.grid)
    out["abs_dif"] = out["abs_dir"]
    for accumulate in (False, True):
        ws = buffered(df, brick, 192 << 20)
        r.trace(df, 35.0, 20.0, n, 7, workspace=ws, out=out, accumulate=accumulate, **kw)
        assert used(df, brick, ws)
        assert torch.equal(out["abs_dir"], (ref["abs_dir"] + ref["abs_dif"]) * (2 if accumulate else 1))


def test_majorants_that_fill_the_lds():
    """39900 majorants in LDS on request, beside the tracing kernel's own: no
    room for another 256 bytes."""
    df, brick, n = fields((76, 84, 200)), (4, 4, 2), 1 << 22
    kw = dict(brick=brick, diffuse_fraction=0.1, lds_majorant=1)
    ref = r.trace(df, 35.0, 20.0, n, 7, workspace=plain(df, brick), **kw)
    ws = buffered(df, brick, 256 << 20)
    got = r.trace(df, 35.0, 20.0, n, 7, workspace=ws, **kw)
    same(got, ref)
    assert used(df, brick, ws)


# 128 bins, 129 with a ragged last one, 1344 (beyond the line of 1280)
@pytest.mark.parametrize("shape,brick,photons", [((128, 64, 128), (8, 8, 8), (1 << 22) + 12345),
                                                 ((110, 99, 97), (5, 3, 1), (1 << 22) + 1), ((256, 256, 168), (8, 8, 8), 1 << 23)])
@pytest.mark.parametrize("kw", [dict(), dict(merge=False), dict(lds_majorant=-1), dict(sobol_entry=True, photon_offset=77),
                                dict(pool_photons=64, refill_lanes=64, max_walk=1)], ids=lambda k: "-".join(k) or "plain")
def test_options_through_the_buffer(shape, brick, photons, kw):
    """Every option of a trace, with the fewest tiles, one more, and many; then
    added to what is there."""
    df = fields(shape)
    opt = r.options(brick=brick)
    kw = dict(kw, brick=brick, diffuse_fraction=0.2)
    ref = r.trace(df, 35.0, 20.0, photons, 7, workspace=plain(df, brick), **kw)
    least = spare_for(df.grid, opt, photons, 512 * LANES, 1)
    for spare in (least, least + 140000, 8 * least):
        print("options case", shape, photons, spare, flush=True)
        ws = buffered(df, brick, spare)
        got = r.trace(df, 35.0, 20.0, photons, 7, workspace=ws, **kw)
        same(got, ref)
        assert used(df, brick, ws)
    more = dict(kw, photon_offset=photons + 1000)
    r.trace(df, 35.0, 20.0, photons, 8, workspace=plain(df, brick), out=ref, accumulate=True, **more)
    r.trace(df, 35.0, 20.0, photons, 8, workspace=ws, out=got, accumulate=True, **more)
    same(got, ref)


def test_capped_photons_and_sums_beyond_32_bits():
    """Photons stopped by max_iters while the buffer fills several times, and cells
    whose sum in one round passes 32 bits."""
    grid, brick, n = syn.Grid(128, 64, 128, 50.0, 50.0, 50.0), (8, 8, 8), 1 << 24
    df = r.DeviceFields.from_host(syn.uniform_fields(grid, 0.02, 0.01, 0.3, 0.5, 0.3))
    kw = dict(brick=brick, max_iters=9, rr_threshold=0.05)
    spare = spare_for(grid, r.options(brick=brick), n, 512 * LANES, 1)
    ref = r.trace(df, 10.0, 0.0, n, 5, workspace=plain(df, brick), **kw)
    ws = buffered(df, brick, spare)
    got = r.trace(df, 10.0, 0.0, n, 5, workspace=ws, **kw)
    same(got, ref)
    assert used(df, brick, ws)
    assert int(ref["stats"][r.STATS.index("capped")]) > 0
    assert int(ref["abs_dir"].max()) > 1 << 36 and int((ref["abs_dir"] + ref["abs_dif"]).sum() >> 31) > 0


def test_captured_in_a_graph():
    """The rounds recorded in a graph: each replay is the eager call, whatever the
    workspace and the outputs hold and the device does in between."""
    df, brick, n = fields((128, 64, 128)), (8, 8, 8), 1 << 22
    kw = dict(brick=brick, diffuse_fraction=0.1)
    ref = r.trace(df, 35.0, 20.0, n, 7, workspace=plain(df, brick), **kw)
    ws, out = buffered(df, brick, 256 << 20), r.alloc_tallies(df.grid)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        r.trace(df, 35.0, 20.0, n, 7, workspace=ws, out=out, **kw)
    out.pop("photons")
    for k in range(4):
        ws.fill_(0xff if k & 1 else 0)
        for v in out.values():
            v.fill_(k)
        graph.replay()
        same(out, ref)
        other = r.trace(df, 35.0, 20.0, 1 << 16, 9, workspace=plain(df, brick), **kw)
        assert int(other["stats"][0]) == 1 << 16
