"""The photon schedule of totals that no launch has (2^33 photons and more),
slot by slot against integers of any size."""
import pytest

from paper_2208_05247_amd import rt3d
from paper_2208_05247_amd.synthetic import Grid


def slot(nx, ny, counts, offs, tile, po, s):
    """(g-point, id, column) of slot s, as rt3d.h defines the schedule."""
    ncol, (tx, ty) = nx * ny, tile
    passes = [c // ncol for c in counts]
    full = sum(passes) * ncol
    if s < full:
        t, rem = divmod(s, tx * ty * sum(passes))
        f, u = divmod(rem, tx * ty)
        n = 0
        while f >= passes[n]:
            f -= passes[n]
            n += 1
        col = (t // (nx // tx) * ty + u // tx) * nx + t % (nx // tx) * tx + u % tx
        k = (col - offs[n] - po) % ncol + f * ncol
    else:
        q, n = s - full, 0
        while q >= counts[n] % ncol:
            q -= counts[n] % ncol
            n += 1
        k = passes[n] * ncol + q
        col = (po + k + offs[n]) % ncol
    return n, po + k, col


@pytest.mark.parametrize("nx,ny,tile,counts,offs", [
    (1, 1, (1, 1), [(1 << 57) + 5], [0]), (3, 1, (1, 1), [(1 << 60) + 1], [2]), (8, 6, (4, 3), [(1 << 33) - 1], [47]),
    (8, 6, (4, 3), [(1 << 33) + 7, 3, 1 << 40], [5, 0, 47]), (7, 5, (7, 1), [1 << 52, (1 << 53) + 1], [34, 0]),
    (1000, 999, (20, 27), [(1 << 62) + 12345, (1 << 61) + 1], [998999, 3])])
@pytest.mark.parametrize("po", [0, (1 << 40) + 3])
def test_any_total(nx, ny, tile, counts, offs, po):
    opt = rt3d.options(brick=(1, 1, 1), tile=tile, photon_offset=po)
    total = sum(counts)
    full = sum(c // (nx * ny) for c in counts) * nx * ny
    at = {0, total - 1, full - 1, min(full, total - 1), (1 << 33) - 2, (1 << 33) - 1, 1 << 33, (1 << 33) + 1}
    at |= {total * i // 37 for i in range(37)} | {total // 2 + i for i in range(-3, 4)}
    for s in sorted(a for a in at if 0 <= a < total):
        gp, ids, cols = rt3d.schedule_slots(Grid(nx, ny, 4, 10.0, 10.0, 10.0), counts, offs, opt, first_slot=s, n=1)
        assert (int(gp[0]), int(ids[0]), int(cols[0])) == slot(nx, ny, counts, offs, tile, po, s), s
