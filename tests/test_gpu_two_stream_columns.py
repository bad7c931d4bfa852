"""The two-stream column on both sides of the rule that gives a column a lane
or a workgroup: many columns, the most that a workgroup each can launch and one
more.  Against the adding method on the host (FP64, the bound of the column
lengths' test: 1e-11 of the flux at the top) for the first, last and some other
columns."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import two_stream_adding as ref  # noqa: E402
from paper_2208_05247_amd import rt3d  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nlay,nc", [
    (1, 8192), (1, 8193), (12, 8193), (16, 10000), (16, 10001), (16, 60001), (24, 12289), (24, 49153), (100, 16385), (100, 40961), (352, 16385),
    (400, 16384), (400, 16385), (480, 12500), (480, 12501), (1024, 5859), (1024, 5860), (1, (1 << 25) - 1), (1, 1 << 25)])
def test_many_columns(nlay, nc):
    g = torch.Generator(device="cuda").manual_seed(nlay + nc)
    u = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float64)
    tau = torch.exp(u(nc, nlay) * 14.0 - 13.0) / nlay ** 0.5
    ssa, asy, alb, ftoa = u(nc, nlay) * 0.949 + 0.05, u(nc, nlay) * 0.8, u(nc) * 0.9, u(nc) * 1.9 + 0.1
    mu0, tod = 0.6, nlay // 2
    print("columns", nlay, nc, flush=True)
    out = rt3d.two_stream(tau, ssa, asy, alb, mu0, tod, flux_toa=ftoa)
    for c in sorted({0, 1, 63, 64, nc // 2, nc - 65, nc - 2, nc - 1}):
        s, d, up = ref.column(*(a[c].cpu().numpy() for a in (tau, ssa, asy)), mu0, alb[c].item(), ftoa[c].item())
        top = abs(s[0])
        for name, want in (("dir", s), ("dn_dif", d), ("up", up)):
            assert np.abs(out[name][c].cpu().numpy() - want).max() <= 1e-11 * top, (name, c)
        assert abs(out["tod_flux"][c].item() - (s[tod] + d[tod])) <= 1e-11 * top
    assert bool(torch.isfinite(out["up"]).all()) and bool((out["dir"][:, 0] == mu0 * ftoa).all())
