"""Workloads of the tracer and the denoiser, called through the public Python
entry points as a user's program calls them.

Twelve listed cases span the range in use: single-g-point traces from one
latency-bound batch of 2**14 photons to the 256x256x128 LES-shaped field,
batched 112-g-point traces from a training scene to the 1024x1024x128 domain,
the steps around them (normalisation, two-stream entry flux), and the learned
denoiser: whole inference, one training pass, single layers forward and
backward, the optimiser update.  ``draw`` takes further sizes of the same
ranges, odd ones among them.
"""
import math

import numpy as np
import torch

from paper_2208_05247_amd import denoise as dn
from paper_2208_05247_amd import experiment as ex
from paper_2208_05247_amd import rt3d
from paper_2208_05247_amd import synthetic as syn


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # one 2**14-photon batch on a 32x32x64 field (error bars from many
        # small batches, the smoke check): launches and latency count
        {"name": "trace_small", "kind": "trace", "nx": 32, "ny": 32, "nz": 64, "dx": 100.0, "dz": 50.0,
         "bx": 4, "by": 4, "bz": 4, "photons": 1 << 14, "sza": 30.0, "diffuse": 0.0, "sobol": False,
         "accumulate": False},
        # odd grid, majorant cells that divide it, part of the light diffuse,
        # scrambled-Sobol entry, added to the tallies of earlier calls
        {"name": "trace_ragged", "kind": "trace", "nx": 90, "ny": 66, "nz": 50, "dx": 50.0, "dz": 40.0,
         "bx": 5, "by": 6, "bz": 5, "photons": 1500007, "sza": 52.5, "diffuse": 0.15, "sobol": True,
         "accumulate": True},
        # the LES-shaped cumulus field of the benchmark, 1024 photons a column
        {"name": "trace_les", "kind": "trace", "nx": 256, "ny": 256, "nz": 128, "dx": 50.0, "dz": 25.0,
         "bx": 8, "by": 8, "bz": 8, "photons": 1 << 26, "sza": 45.0, "diffuse": 0.0, "sobol": False,
         "accumulate": False},
        # one noisy input of a denoiser training scene: 112 g-points in one
        # launch, diffuse share per g-point, 256 photons a column
        {"name": "batched_scene", "kind": "batched", "nx": 128, "ny": 128, "nz": 128, "dx": 25.0, "dz": 20.0,
         "ngp": 112, "per_col": 256.0, "sza": 40.0},
        # the large domain with every g-point, 128 photons a column (the low
        # end of what the denoiser takes as input)
        {"name": "batched_large", "kind": "batched", "nx": 1024, "ny": 1024, "nz": 128, "dx": 25.0, "dz": 20.0,
         "ngp": 112, "per_col": 128.0, "sza": 60.0},
        # tallies of a 512x512x96 domain into heating rates and fluxes
        {"name": "finalize_mid", "kind": "finalize", "nx": 512, "ny": 512, "nz": 96, "dx": 50.0, "dz": 32.0},
        # entry flux of 112 g-points: 32 layers above the domain, 128 in it
        {"name": "two_stream", "kind": "two_stream", "cols": 112, "nlay": 160, "tod": 32, "mu0": 0.5},
        # whole inference with the committed weights on a small odd field
        {"name": "denoise_small", "kind": "denoise", "D": 40, "H": 56, "W": 72},
        # and on the large domain (128 levels of 1024x1024)
        {"name": "denoise_large", "kind": "denoise", "D": 128, "H": 1024, "W": 1024},
        # forward, loss and backward on one 128**3 training scene
        {"name": "train_pass", "kind": "train", "D": 128, "H": 128, "W": 128},
        # the finest decoder layer's input concatenation on a ragged grid:
        # first input at half resolution, second at full
        {"name": "decoder_layer", "kind": "conv", "D": 44, "H": 90, "W": 118, "c1": 128, "c2": 64, "cout": 64, "up": True},
        # weight and bias gradient of an encoder layer at half resolution
        {"name": "layer_wgrad", "kind": "wgrad", "D": 64, "H": 60, "W": 52, "c1": 32, "c2": 0, "cout": 64},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _side(rng, lo, hi, step):
    """A multiple of step, log-uniform in [lo, hi]."""
    return step * max(1, round(_log(rng, lo, hi) / step))


def draw(rng):
    kind = rng.choice(["trace", "trace", "batched", "finalize", "two_stream", "denoise", "train", "conv", "wgrad"])
    if kind == "trace":
        bx, by, bz = rng.choice([(8, 8, 8), (4, 4, 4), (5, 6, 5), (8, 4, 2), (7, 3, 9)])
        nx, ny, nz = _side(rng, 24, 300, bx), _side(rng, 24, 300, by), _side(rng, 24, 140, bz)
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "dx": rng.choice([25.0, 50.0, 100.0]),
                "dz": rng.choice([20.0, 25.0, 50.0]), "bx": bx, "by": by, "bz": bz,
                "photons": int(_log(rng, 1 << 12, 1 << 25)), "sza": rng.uniform(0.0, 70.0),
                "diffuse": rng.choice([0.0, 0.0, 0.2, 1.0]), "sobol": rng.random() < 0.3,
                "accumulate": rng.random() < 0.3}
    if kind == "batched":
        nx, ny, nz = _side(rng, 32, 512, 8), _side(rng, 32, 512, 8), _side(rng, 32, 128, 8)
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "dx": rng.choice([25.0, 50.0]),
                "dz": rng.choice([20.0, 32.0]), "ngp": rng.choice([1, 7, 16, 64, 112, 224]),
                "per_col": min(_log(rng, 8, 768), (1 << 26) / (nx * ny)), "sza": rng.uniform(0.0, 65.0)}
    if kind == "finalize":
        return {"kind": kind, "nx": int(_log(rng, 31, 512)), "ny": int(_log(rng, 31, 512)),
                "nz": int(_log(rng, 16, 130)), "dx": 50.0, "dz": 25.0}
    if kind == "two_stream":
        nlay = int(_log(rng, 16, 300))
        return {"kind": kind, "cols": int(_log(rng, 1, 4096)), "nlay": nlay, "tod": rng.randrange(nlay + 1),
                "mu0": rng.uniform(0.05, 1.0)}
    if kind == "denoise":
        return {"kind": kind, "D": _side(rng, 16, 128, 8), "H": _side(rng, 16, 256, 8), "W": _side(rng, 16, 256, 8)}
    if kind == "train":
        return {"kind": kind, "D": _side(rng, 16, 128, 8), "H": _side(rng, 16, 128, 8), "W": _side(rng, 16, 128, 8)}
    if kind == "conv":
        c1, c2, cout, up = rng.choice([(32, 0, 64, False), (64, 0, 128, False), (128, 0, 256, False),
                                       (256, 128, 128, True), (128, 64, 64, True), (64, 32, 32, True),
                                       (64, 32, 32, False)])
        s = 2 if up else 1
        return {"kind": kind, "D": _side(rng, 8, 64, s), "H": _side(rng, 10, 100, s), "W": _side(rng, 10, 140, s),
                "c1": c1, "c2": c2, "cout": cout, "up": up}
    c1, c2, cout = rng.choice([(16, 0, 32), (32, 0, 64), (64, 0, 128), (128, 0, 256), (256, 128, 128), (128, 64, 64),
                               (64, 32, 32)])
    return {"kind": kind, "D": int(_log(rng, 4, 40)), "H": int(_log(rng, 6, 60)), "W": int(_log(rng, 6, 80)),
            "c1": c1, "c2": c2, "cout": cout}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _grid(c):
    return syn.Grid(c["nx"], c["ny"], c["nz"], c["dx"], c["dx"], c["dz"])


def _cloud(grid, seed):
    """Cumulus extinction (m^-1) on the device: truncated Gaussian blobs
    between 27 % and 98 % of the domain height, 200 per 12.8 x 12.8 km (at
    least 4), amplitude log-normal around 0.02, radius 150-400 m (less in a
    shallow domain), periodic in x and y."""
    r = np.random.default_rng(int(seed))
    lx, ly, h = grid.nx * grid.dx, grid.ny * grid.dy, grid.nz * grid.dz
    n = max(4, int(round(200 * lx * ly / 12800.0 ** 2)))
    k = torch.zeros(grid.shape3, device="cuda")
    lo, hi = 0.27 * h, 0.98 * h
    for _ in range(n):
        sig = min(r.uniform(150.0, 400.0), 0.2 * h)
        cx, cy, cz = r.uniform(0, lx), r.uniform(0, ly), r.uniform(lo + sig, hi - sig)
        amp = 0.02 * math.exp(0.5 * r.standard_normal())
        index, square = [], []
        for centre, d, m, wraps in ((cz, grid.dz, grid.nz, False), (cy, grid.dy, grid.ny, True),
                                    (cx, grid.dx, grid.nx, True)):
            first, last = math.floor((centre - 2 * sig) / d), math.ceil((centre + 2 * sig) / d)
            if wraps:
                last = min(last, first + m - 1)
            i = np.arange(first, last + 1)
            if not wraps:
                i = i[(i >= 0) & (i < m)]
            square.append(torch.from_numpy(((i + 0.5) * d - centre) ** 2).float().cuda())
            index.append(torch.from_numpy(i % m).cuda())
        r2 = square[0][:, None, None] + square[1][None, :, None] + square[2][None, None, :]
        k[index[0][:, None, None], index[1][None, :, None], index[2][None, None, :]] += torch.where(
            r2 <= 4 * sig * sig, amp * torch.exp(r2 / (-2 * sig * sig)), 0.0)
    z = (torch.arange(grid.nz, device="cuda") + 0.5) * grid.dz
    k[(z < lo) | (z > hi)] = 0.0
    return k


def _heating(D, H, W, seed):
    """Noisy heating-rate fields as low-photon tracing gives them (most cells
    small, heavy tail, many empty) with the gray extinction and absorption of
    a cloud field, and the noise-free heating."""
    grid = syn.Grid(W, H, D, 25.0, 25.0, 20.0)
    kc = _cloud(grid, seed)
    g = _gen(seed)
    depth = torch.linspace(1.0, 0.3, D, device="cuda").flip(0)[:, None, None]
    clean_dir = 4.0 * depth * (1.0 + 30.0 * kc) * torch.exp(-10.0 * kc)
    clean_dif = 1.5 * depth * (1.0 + 60.0 * kc)
    noise = lambda p: torch.empty(p.shape, device="cuda").exponential_(generator=g) * \
        (torch.rand(p.shape, generator=g, device="cuda") < 0.6) / 0.6
    return ((clean_dir * noise(clean_dir)).contiguous(), (clean_dif * noise(clean_dif)).contiguous(),
            (kc + 2e-4).contiguous(), (kc * 5e-4 + 1e-5).contiguous(), clean_dir, clean_dif)


def _conv_inputs(c, seed):
    g = _gen(seed)
    D, H, W = c["D"], c["H"], c["W"]
    s = 2 if c.get("up") else 1
    act = lambda *shape: torch.relu(torch.randn(*shape, generator=g, device="cuda")).to(torch.bfloat16)
    x1 = act(D // s, H // s, W // s, c["c1"])
    x2 = act(D, H, W, c["c2"]) if c["c2"] else None
    cin = c["c1"] + c["c2"]
    w = (torch.randn(c["cout"], 27, cin, generator=g, device="cuda") * math.sqrt(2.0 / (27 * cin))).to(torch.bfloat16)
    b = torch.randn(c["cout"], generator=g, device="cuda") * 0.1
    return x1, x2, w, b, g


def _net(seed):
    """A network as in the middle of training: every layer passes gradient."""
    net = dn.Denoiser(base=32, seed=int(seed))
    g = torch.Generator().manual_seed(int(seed) + 1)
    net.p["head"][:dn.NOUT] = (torch.randn(dn.NOUT, *net.p["head"].shape[1:], generator=g) * 0.1).cuda()
    for k in net.bias:
        net.bias[k].copy_((torch.randn(net.bias[k].shape, generator=g) * 0.05).cuda())
        net.pb[k].copy_(net.p[k].to(torch.bfloat16))
    return net


def _two_stream_inputs(c, seed):
    g = _gen(seed)
    n, m = c["cols"], c["nlay"]
    f64 = dict(generator=g, device="cuda", dtype=torch.float64)
    # column optical depth log-uniform over the g-points, thinning upwards
    col = torch.exp(math.log(1e-3) + math.log(5e4) * torch.rand(n, 1, **f64))
    shape = torch.exp(torch.linspace(-6.0, 0.0, m, device="cuda", dtype=torch.float64))[None, :]
    tau = (col * shape / shape.sum()).contiguous()
    ssa = (0.2 + 0.8 * torch.rand(n, 1, **f64)).expand(n, m).contiguous()
    return {"tau": tau, "ssa": ssa, "g": torch.zeros_like(tau), "albedo": 0.1 + 0.2 * torch.rand(n, **f64),
            "flux_toa": torch.rand(n, **f64) + 1e-3}


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "trace":
        grid = _grid(c)
        kc = _cloud(grid, seed)
        z = (torch.arange(grid.nz, device="cuda") + 0.5) * grid.dz
        kg = (1e-5 * torch.exp(z / -8000.0))[:, None, None].expand(grid.shape3)
        ke = kg + kc
        df = rt3d.DeviceFields(grid, ke.contiguous(), kc, ((0.9 * kg + 0.9995 * kc) / ke).clamp(0, 1).contiguous(),
                               torch.where(kc > 0, 0.86, 0.0).contiguous(),
                               0.1 + 0.2 * torch.rand(grid.shape2, generator=_gen(seed), device="cuda"))
        brick = (c["bx"], c["by"], c["bz"])
        out = rt3d.alloc_tallies(grid)
        if c["accumulate"]:
            for t in out.values():
                t.zero_()
        ws = rt3d.alloc_workspace(rt3d.workspace_size(grid, rt3d.options(brick=brick)))
        return {"case": c, "df": df, "brick": brick, "out": out, "ws": ws, "seed": int(seed)}
    if kind == "batched":
        grid = _grid(c)
        kc = _cloud(grid, seed)
        cloudy = kc > 0
        r = np.random.default_rng(int(seed))
        kg, og, shares = syn.gpoint_set(grid, c["ngp"], r)
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
        dm = rt3d.DeviceBatchedMedium(grid, up(kg), up(og), kc, torch.where(cloudy, 0.9995, 0.0).contiguous(),
                                      torch.where(cloudy, 0.86, 0.0).contiguous(),
                                      0.1 + 0.2 * torch.rand(grid.shape2, generator=_gen(seed), device="cuda"))
        counts = r.multinomial(max(1, int(c["per_col"] * grid.ncol)), shares).astype(np.uint64)
        fd = up(r.uniform(0.02, 0.3, c["ngp"]))
        ws = rt3d.alloc_workspace(rt3d.workspace_size_batched(grid, c["ngp"], rt3d.options()))
        return {"case": c, "dm": dm, "counts": counts, "fd": fd, "out": rt3d.alloc_tallies(grid), "ws": ws,
                "seed": int(seed)}
    if kind == "finalize":
        grid = _grid(c)
        g = _gen(seed)
        raw = {}
        for n, t in rt3d.alloc_tallies(grid).items():
            # 256 photons a column: deposits of a few 2^-31 units to some weights
            raw[n] = (torch.empty(t.shape, device="cuda").exponential_(generator=g) * 2.0 ** 29).to(torch.int64)
        return {"case": c, "grid": grid, "raw": raw, "photons": 256 * grid.ncol, "scale": ex.layer_scale(grid)}
    if kind == "two_stream":
        return {"case": c, **_two_stream_inputs(c, seed)}
    if kind == "denoise":
        net, _ = ex.load_committed_denoiser()
        return {"case": c, "net": net, "fields": _heating(c["D"], c["H"], c["W"], seed)[:4]}
    if kind == "train":
        net = _net(seed)
        hd, hf, ke, ka, cd, cf = _heating(c["D"], c["H"], c["W"], seed)
        s = dn.field_scale(hd, hf)
        feat, base = dn.features(hd, hf, ke, ka, 20.0, s)
        return {"case": c, "net": net, "feat": feat, "base": base,
                "target": torch.stack([cd / s, cf / s], dim=-1).float().contiguous()}
    if kind == "conv":
        x1, x2, w, b, _ = _conv_inputs(c, seed)
        return {"case": c, "x1": x1, "x2": x2, "w": w, "b": b,
                "y": dn.bf16_empty(c["D"], c["H"], c["W"], c["cout"])}
    x1, x2, w, _, g = _conv_inputs(c, seed)
    dz = torch.randn(c["D"], c["H"], c["W"], c["cout"], generator=g, device="cuda").to(torch.bfloat16)
    ws = torch.empty(dn.wgrad_workspace_size(x1, x2, c["cout"], 3), dtype=torch.uint8, device="cuda")
    return {"case": c, "x1": x1, "x2": x2, "dz": dz, "ws": ws, "dw": torch.empty(w.shape, device="cuda"),
            "db": torch.empty(c["cout"], device="cuda")}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "trace":
        return rt3d.trace(s["df"], c["sza"], 30.0, c["photons"], s["seed"], brick=s["brick"],
                          diffuse_fraction=c["diffuse"], sobol_entry=c["sobol"], accumulate=c["accumulate"],
                          out=s["out"], workspace=s["ws"])
    if kind == "batched":
        return rt3d.trace_batched(s["dm"], c["sza"], 30.0, s["counts"], s["seed"], gpoint_diffuse=s["fd"],
                                  out=s["out"], workspace=s["ws"])
    if kind == "finalize":
        return rt3d.finalize(s["grid"], s["raw"], s["photons"], layer_scale=s["scale"], flux_scale=1000.0)
    if kind == "two_stream":
        return rt3d.two_stream(s["tau"], s["ssa"], s["g"], s["albedo"], c["mu0"], c["tod"], flux_toa=s["flux_toa"])
    if kind == "denoise":
        return dn.denoise(s["net"], *s["fields"], 20.0)
    if kind == "train":
        # a training step up to the optimiser update (whose moments would
        # make the next pass on the same state another problem)
        net = s["net"]
        out = net.forward(s["feat"], keep=True)
        pred, dout, loss = dn.mse(out, s["base"], s["target"], want_grad=True)
        net.backward(dout)
        return {"loss": loss, "pred": pred, "g": net.g, "gbias": net.gbias}
    if kind == "conv":
        dn.conv_fwd(s["x1"], s["x2"], s["w"], s["b"], True, c["cout"], 3, y1=s["y"], up1=c["up"])
        return s["y"]
    s["dw"].zero_()
    s["db"].zero_()
    dn.conv_wgrad(s["x1"], s["x2"], s["dz"], c["cout"], 3, s["dw"], s["db"], workspace=s["ws"])
    return s["dw"], s["db"]


# Flops of the network per full-resolution voxel: 27 taps x input channels x
# output channels x 2, by level (4 real channels in the first layer)
_NET = 2 * (27 * (4 * 32 + 32 * 64 / 8 + 64 * 128 / 64 + 128 * 256 / 512 + 384 * 128 / 64 + 192 * 64 / 8 + 96 * 32)
            + 32 * 2)


def work(case):
    c, kind = case, case["kind"]
    if kind in ("trace", "batched"):
        cells, cols = c["nx"] * c["ny"] * c["nz"], c["nx"] * c["ny"]
        fields = 16 if kind == "trace" else 12
        photons = c["photons"] if kind == "trace" else c["per_col"] * cols
        # about 30 events a photon (collisions and cell crossings), about
        # 200 operations an event with its random numbers
        return {"bytes": cells * (fields + 16 * (2 if c.get("accumulate") else 1)) + cols * 36, "flops": photons * 30 * 200}
    if kind == "finalize":
        return {"bytes": 12 * (2 * c["nx"] * c["ny"] * c["nz"] + 4 * c["nx"] * c["ny"]), "flops": 0}
    if kind == "two_stream":
        n = c["cols"] * c["nlay"]
        return {"bytes": 48 * n, "flops": 300 * n}
    if kind == "conv":
        v, cin = c["D"] * c["H"] * c["W"], c["c1"] + c["c2"]
        return {"bytes": 2 * v * (c["c1"] / (8 if c["up"] else 1) + c["c2"] + c["cout"]) + 54 * cin * c["cout"],
                "flops": 54 * v * cin * c["cout"]}
    if kind == "wgrad":
        v, cin = c["D"] * c["H"] * c["W"], c["c1"] + c["c2"]
        return {"bytes": 2 * v * (cin + c["cout"]) + 108 * cin * c["cout"], "flops": 54 * v * cin * c["cout"]}
    v = c["D"] * c["H"] * c["W"]
    if kind == "denoise":
        return {"bytes": 24 * v, "flops": _NET * v}
    # kept activations written and read back: 32 channels and a 64- and
    # 32-channel decoder input at full resolution, the coarser levels 1/8 each
    return {"bytes": v * (32 + 8 * 3 + 2 * 2 * (32 + 32 + 64) * 8 / 7), "flops": 3 * _NET * v}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def _conv64(x, w, b=None):
    """3x3x3 (or 1x1x1) zero-padded convolution, [D][H][W][C] by [O][taps][C]."""
    k = round(w.shape[1] ** (1 / 3))
    D, H, W, _ = x.shape
    p = k // 2
    xp = torch.nn.functional.pad(x, (0, 0, p, p, p, p, p, p))
    y = 0
    for t in range(k ** 3):
        z, r, q = t // (k * k), (t // k) % k, t % k
        y = y + (xp[z:z + D, r:r + H, q:q + W].reshape(-1, x.shape[3]) @ w[:, t].t()).reshape(D, H, W, -1)
    return y if b is None else y + b


def _up64(x):
    return x.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)


def _pool64(x):
    D, H, W, C = x.shape
    return x.reshape(D // 2, 2, H // 2, 2, W // 2, 2, C).mean(dim=(1, 3, 5))


def _net64(x, w, b):
    r = lambda n, *xs: torch.relu(_conv64(torch.cat(xs, 3), w[n], b[n]))
    e0 = r("e0", x)
    e1 = r("e1", _pool64(e0))
    e2 = r("e2", _pool64(e1))
    d = r("d2", _up64(r("b", _pool64(e2))), e2)
    d = r("d0", _up64(r("d1", _up64(d), e1)), e0)
    return _conv64(d, w["head"], b["head"])


def _two_stream64(s, c):
    """Adding method for all columns at once (practical improved flux method
    coefficients), CPU."""
    h = lambda k: s[k].cpu()
    tau, w, g, alb, mu = h("tau"), h("ssa"), h("g"), h("albedo"), c["mu0"]
    n, m = tau.shape
    g1, g2 = 0.25 * (8 - w * (5 + 3 * g)), 0.75 * w * (1 - g)
    k = ((g1 - g2) * (g1 + g2)).clamp(min=0).sqrt().clamp(min=1e-12)
    e, x = torch.exp(-k * tau), -torch.expm1(-2 * k * tau)
    den = k * (1 + e * e) + g1 * x
    R, T = g2 * x / den, 2 * k * e / den

    def direct(mu):
        g3 = 0.25 * (2 - 3 * mu * g)
        g4, d, tb = 1 - g3, 1 - k * k * mu * mu, torch.exp(-tau / mu)
        a = w * (g3 * (1 - g1 * mu) - g2 * g4 * mu) / d
        q = -w * (g4 * (1 + g1 * mu) + g2 * g3 * mu) / d
        return a - R * q - T * a * tb, q * tb - T * q - R * a * tb

    near = (1 - k * k * mu * mu).abs() < 1e-5
    at, lo, hi = direct(mu), direct(mu * (1 - 1e-5)), direct(mu * (1 + 1e-5))
    Rd, Td = (torch.where(near, 0.5 * (p + q), v) for v, p, q in zip(at, lo, hi))
    S = torch.empty(n, m + 1, dtype=torch.float64)
    S[:, 0] = h("flux_toa") * mu
    for i in range(m):
        S[:, i + 1] = S[:, i] * torch.exp(-tau[:, i] / mu)
    rb, q = torch.empty_like(S), torch.empty_like(S)
    rb[:, m], q[:, m] = alb, alb * S[:, m]
    for i in range(m - 1, -1, -1):
        f = 1 / (1 - R[:, i] * rb[:, i + 1])
        q[:, i] = Rd[:, i] * S[:, i] + T[:, i] * (q[:, i + 1] + rb[:, i + 1] * Td[:, i] * S[:, i]) * f
        rb[:, i] = R[:, i] + T[:, i] ** 2 * rb[:, i + 1] * f
    D, U = torch.zeros_like(S), torch.empty_like(S)
    U[:, 0] = q[:, 0]
    for i in range(m):
        D[:, i + 1] = (T[:, i] * D[:, i] + Td[:, i] * S[:, i] + R[:, i] * q[:, i + 1]) / (1 - R[:, i] * rb[:, i + 1])
        U[:, i + 1] = rb[:, i + 1] * D[:, i + 1] + q[:, i + 1]
    tot = S[:, c["tod"]] + D[:, c["tod"]]
    return {"dir": S, "dn_dif": D, "up": U, "tod_flux": tot, "tod_diffuse_fraction": D[:, c["tod"]] / tot}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("trace", "batched"):
        return None  # whole numbers of one random sequence
    if kind in ("denoise", "train") and c["D"] * c["H"] * c["W"] > 1 << 20:
        return None  # too long in 64 bits
    s = prepare(case, seed)
    if kind == "finalize":
        norm = s["grid"].ncol / (s["photons"] * 2.0 ** 31)
        return {n: s["raw"][n].double() * (norm * s["scale"][:, None, None] if n in rt3d.TALLY3 else norm * 1000.0)
                for n in rt3d.TALLY3 + rt3d.TALLY2}
    if kind == "two_stream":
        return _two_stream64(s, c)
    if kind == "conv":
        x = _up64(s["x1"].double()) if c["up"] else s["x1"].double()
        x = x if s["x2"] is None else torch.cat([x, s["x2"].double()], 3)
        return torch.relu(_conv64(x, s["w"].double(), s["b"].double()))
    if kind == "wgrad":
        x = s["x1"] if s["x2"] is None else torch.cat([s["x1"], s["x2"]], 3)
        D, H, W, _ = x.shape
        xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1, 1, 1))
        dz = s["dz"].double().reshape(-1, c["cout"]).t().contiguous()
        dw = torch.stack([dz @ xp[t // 9:t // 9 + D, (t // 3) % 3:(t // 3) % 3 + H, t % 3:t % 3 + W].reshape(-1, x.shape[3])
                          for t in range(27)], dim=1)
        return dw, dz.sum(dim=1)
    net = s["net"]
    w = {k: v.double() for k, v in net.pb.items()}
    b = {k: v.double() for k, v in net.bias.items()}
    if kind == "denoise":
        hd, hf, ke, ka = (t.double() for t in s["fields"])
        sc = float((hd.mean() + hf.mean()) / 2)
        x = torch.stack([hd / sc, hf / sc, torch.log1p(20 * ke * 20.0), torch.log1p(200 * ka * 20.0)], 3)
        w["e0"] = w["e0"][:, :, :4]
        y = _net64(x, w, b)
        return tuple((y[..., i] + h / sc).clamp(min=0) * sc for i, h in ((0, hd), (1, hf)))
    for t in (*w.values(), *b.values()):
        t.requires_grad_(True)
    pred = _net64(s["feat"].double(), w, b)[..., :dn.NOUT] + s["base"].double()
    loss = ((pred - s["target"].double()) ** 2).mean()
    loss.backward()
    return {"loss": loss.detach().reshape(1), "pred": pred.detach(), "g": {k: v.grad for k, v in w.items()},
            "gbias": {k: v.grad for k, v in b.items()}}
