"""How much more than the needed workspace is allocated for the deposit buffer:
nothing for grids that the library has no buffer for, nor by a call that does
not use it."""
import pytest

from paper_2208_05247_amd import rt3d as r
from paper_2208_05247_amd.synthetic import Grid


@pytest.mark.parametrize("shape,buffered", [((32, 32, 64), False), ((128, 64, 127), False), ((128, 64, 128), True),
                                            ((256, 256, 128), True), ((256, 256, 256), True), ((256, 256, 264), False)])
def test_spare(shape, buffered):
    grid = Grid(*shape, 50.0, 40.0, 30.0)
    opt = r.options(brick=(8, 8, 1))
    size = r.workspace_size(grid, opt)
    spare = getattr(size, "spare", 0)
    assert spare == (max(8 * size, 192 << 20) if buffered else 0)
    photons = 1 << 23
    # of use exactly where the library takes it, with the lanes of a full launch
    assert (r.deposit_plan(grid, opt, photons, size + spare, 512 * 768)["tiles"] > 0) == buffered
    assert (r.deposit_plan(grid, opt, photons, 4 << 30, 512 * 768)["tiles"] > 0) == buffered
    ws = r.alloc_workspace(r._bytes_for(size, 1 << 22, False), device="cpu")
    assert size + spare <= ws.numel() <= size + spare + 256
    for n, aggregate in (((1 << 22) - 1, False), (1 << 22, True)):
        assert size <= r.alloc_workspace(r._bytes_for(size, n, aggregate), device="cpu").numel() <= size + 256
