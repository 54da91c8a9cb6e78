"""The work whose speed is watched, as a user's program asks for it.

Each case is one pass through the public entry points on synthetic inputs:
  decode   micro-models to voxel grids (values, gradients, records; FP32 and
           2-byte lattices; with and without a plan)
  query    value and gradient at a list of positions in a tiled volume
  rays     the same at the samples of an image's rays
  render   a frame of the volume ray caster
  fitstep  loss and gradient of the fit of control points to samples
  grad4    decode of value and gradient, and its backward pass
  fit      least-squares lattices of sampled blocks
  search   error maps of every lattice size of sampled blocks
exact() repeats a case in 64 bits with torch alone, from the definition of a
clamped tensor-product B-spline.
"""
import math

import numpy as np
import torch

import paper_2409_00184_amd as fa

DEV = "cuda"
ALL, VALUE, GRAD = 15, 1, 14


def listed():
    return [
        # one micro-model, the smallest call there is: latency of a launch
        # and of one block spread over the chip (a viewer that refreshes one block)
        dict(name="decode one model", kind="decode", blocks=1, res="64x64x64", ncp="16", degrees="3",
             out="all", dtype="f32", how="default", field="sines", knots="uniform"),
        # a volume's worth of adaptive micro-models to value and gradient
        # grids, planar channels, the call with no options
        dict(name="decode uneven batch", kind="decode", blocks=512, res="64x64x64", ncp="8,12,16,24,32",
             degrees="2,3", out="all", dtype="f32", how="default", field="sines", knots="uniform"),
        # the same kind of batch through a kept plan into one 16-byte record
        # per voxel (the layout a sampler of value and gradient reads)
        dict(name="decode records by plan", kind="decode", blocks=384, res="64x64x64", ncp="8,12,16,24,32",
             degrees="2,3", out="records", dtype="f32", how="plan", field="sines", knots="uniform"),
        # reconstruction of the values only, on odd grids, lattices of any size
        dict(name="decode odd values", kind="decode", blocks=400, res="61x47x53", ncp="5,9,14,21,30,41",
             degrees="1,2,3", out="value", dtype="f32", how="default", field="sines", knots="uniform"),
        # a large turbulence volume kept in BF16, decoded on the matrix cores
        dict(name="decode bf16 matrix", kind="decode", blocks=512, res="64x64x64", ncp="32", degrees="3",
             out="all", dtype="bf16", how="matrix", field="turbulence", knots="uniform"),
        # particles or probes anywhere in a volume of 16^3 micro-models
        dict(name="query scattered", kind="query", n=4_000_000, cells="16x16x16", ncp_lo=8, ncp_hi=32,
             degree=3, dtype="f32", knots="uniform", order="scattered", empty=0.0),
        # the samples of an image's rays through such a volume
        dict(name="query rays", kind="rays", width=960, height=540, samples=192, cells="16x16x16", ncp_lo=8,
             ncp_hi=32, degree=3, dtype="f32", knots="uniform", empty=0.0),
        # a frame with early termination, as an interactive viewer draws it
        dict(name="render frame", kind="render", width=1280, height=720, samples=512, opacity=0.98,
             cells="16x16x16", ncp_lo=8, ncp_hi=32, degree=3, dtype="f32", knots="uniform", empty=0.0),
        # one iteration of a gradient-based fit to turbulence samples
        dict(name="fit iteration", kind="fitstep", blocks=256, res="64x64x64", ncp="16,24,32", degrees="3"),
        # decode of value and gradient under autograd with a loss on all four
        dict(name="value and gradient fit", kind="grad4", blocks=128, res="64x64x64", ncp="8,12,16,24,32",
             degrees="3"),
        # least-squares encoding of a level's blocks at one lattice size
        dict(name="least-squares fit", kind="fit", blocks=512, res="64x64x64", ncp="32", degrees="3"),
        # the in-level search of the adaptive encoding: every size 5..40
        dict(name="lattice size search", kind="search", blocks=64, res="64x64x64", degree=3, lo=5, hi=40),
    ]


# ------------------------------------------------------------------- draws

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sizes(rng):
    return ",".join(str(n) for n in sorted(rng.sample(range(4, 41), rng.choice((1, 3, 5)))))


def _volume(rng):
    lo = rng.randint(4, 16)
    return dict(cells="x".join(str(rng.choice((3, 5, 8, 12, 16))) for _ in range(3)), ncp_lo=lo,
                ncp_hi=rng.randint(lo, 34), degree=rng.choice((1, 2, 3, 3, 3)),
                dtype=rng.choice(("f32", "f32", "bf16", "f16")), knots=rng.choice(("uniform", "uniform", "jittered")),
                empty=rng.choice((0.0, 0.0, 0.1)))


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "query", "rays", "render", "fitstep", "grad4", "fit", "search"))
    if kind == "decode":
        dtype = rng.choice(("f32", "f32", "bf16", "f16"))
        out = rng.choice(("all", "all", "records", "value", "gradient"))
        res = [rng.choice((16, 32, 48, 64, 64, 80, 96, rng.randint(10, 100))) for _ in range(3)]
        most = max(1, min(512, 500_000_000 // (np.prod(res).item() * (1 if out == "value" else 4))))
        return dict(kind=kind, blocks=min(_log(rng, 1, 512), most), res="x".join(map(str, res)), ncp=_sizes(rng),
                    degrees=rng.choice(("1", "2", "3", "3", "2,3")), out=out, dtype=dtype,
                    how=rng.choice(("default", "plan", "matrix") if dtype != "f32" else ("default", "plan")),
                    field="sines", knots=rng.choice(("uniform", "uniform", "uniform", "jittered")))
    if kind == "query":
        return dict(kind=kind, n=_log(rng, 1000, 4_000_000), order=rng.choice(("scattered", "along rays")), **_volume(rng))
    if kind == "rays":
        return dict(kind=kind, width=rng.randint(60, 900), height=rng.randint(40, 500), samples=rng.randint(20, 190),
                    **_volume(rng))
    if kind == "render":
        return dict(kind=kind, width=rng.randint(100, 1200), height=rng.randint(60, 700), samples=rng.randint(50, 500),
                    opacity=rng.choice((0.95, 0.98, 0.98, 1.0)), **_volume(rng))
    if kind == "search":
        r = rng.choice((16, 24, 32, 48, 64))
        p = rng.choice((2, 3))
        return dict(kind=kind, blocks=_log(rng, 1, 64), res="x".join([str(r)] * 3), degree=p, lo=p + 2,
                    hi=rng.randint(p + 3, r * 5 // 8))
    if kind == "fit":
        res = [rng.choice((32, 48, 64, 64, rng.randint(30, 64))) for _ in range(3)]
        ncp = ",".join(str(n) for n in sorted(rng.sample(range(5, min(res) * 5 // 8 + 1), rng.choice((1, 2, 4)))))
        return dict(kind=kind, blocks=_log(rng, 1, 400), res="x".join(map(str, res)), ncp=ncp,
                    degrees=rng.choice(("2", "3", "3")))
    # fits by gradient; rows that are not whole 16-byte vectors among them
    res = [rng.choice((32, 64, 64, 64, rng.randint(20, 64))) for _ in range(3)]
    return dict(kind=kind, blocks=_log(rng, 1, 256 if kind == "fitstep" else 128), res="x".join(map(str, res)),
                ncp=_sizes(rng), degrees=rng.choice(("2", "3", "3", "2,3")))


# ------------------------------------------------- inputs, with torch alone

def _ints(text, sep="x"):
    return [int(v) for v in text.split(sep)]


def _layout(ncp, deg, jitter, g):
    """Clamped knots (FP32, back to back) and offsets of a batch; interior
    knots moved by up to 15% of a spacing where jitter is set."""
    nb, K = len(ncp), int(ncp.max() + deg.max() + 1)
    j = np.arange(K)[None, None, :]
    n, p = ncp[:, :, None], deg[:, None, None]
    t = np.clip((j - p) / (n - p), 0.0, 1.0)
    if jitter:
        t = t + ((j > p) & (j < n)) * g.uniform(-0.15, 0.15, (nb, 3, K)) / (n - p)
    t = t.astype(np.float32)
    klen = ncp + deg[:, None] + 1
    knots = t[np.arange(K)[None, None, :] < klen[:, :, None]]
    koff = np.concatenate([[0], np.cumsum(klen.sum(1))[:-1]])
    size = ncp.prod(1)
    coff = np.concatenate([[0], np.cumsum((size + 63) // 64 * 64)])
    return t, knots, koff.astype(np.int64), coff[:-1].astype(np.int64), int(coff[-1])


def _sines(ncp, deg, t, coff, total, origin, g):
    """Lattices of a sum of eight sines (up to three cycles per block) taken
    at the Greville points; block b covers [origin_b, origin_b + 1)."""
    k = torch.tensor(g.uniform(-3.0, 3.0, (8, 3)), device=DEV)
    phi = torch.tensor(g.uniform(0.0, 2 * math.pi, 8), device=DEV)
    m = int(ncp.max())
    csum = np.concatenate([np.zeros(t.shape[:2] + (1,)), np.cumsum(t.astype(np.float64), 2)], 2)
    i = np.arange(m)[None, None, :]
    p = deg[:, None, None]
    hi = np.minimum(i + p + 1, t.shape[2])
    xi = (np.take_along_axis(csum, np.broadcast_to(hi, (len(ncp), 3, m)), 2)
          - np.take_along_axis(csum, np.broadcast_to(np.minimum(i + 1, t.shape[2]), (len(ncp), 3, m)), 2)) / p
    x = torch.tensor(xi + np.asarray(origin)[:, :, None], device=DEV)
    n = torch.tensor(ncp, device=DEV)
    off = torch.tensor(coff, device=DEV)
    ctrl = torch.zeros(total, device=DEV)
    ar = torch.arange(m, device=DEV)
    for b0 in range(0, len(ncp), 256):
        s = slice(b0, b0 + 256)
        f = 0.0
        for q in range(8):
            e = torch.exp(2j * math.pi * k[q][None, :, None] * x[s])
            f = f + (e[:, 0, :, None, None] * e[:, 1, None, :, None] * e[:, 2, None, None, :]
                     * torch.exp(1j * phi[q])).imag
        N = n[s]
        inside = ((ar[None, :, None, None] < N[:, 0, None, None, None]) & (ar[None, None, :, None] < N[:, 1, None, None, None])
                  & (ar[None, None, None, :] < N[:, 2, None, None, None]))
        at = (off[s][:, None, None, None] + (ar[None, :, None, None] * N[:, 1, None, None, None] + ar[None, None, :, None])
              * N[:, 2, None, None, None] + ar[None, None, None, :])
        ctrl[at[inside]] = f[inside].float()
    return ctrl


def _turbulence(nb, shape, seed):
    """k^(-5/3) fields (random phases, amplitude |k|^(-11/6)), zero mean and
    unit variance, [nb, *shape] FP32."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    kx, ky = (torch.fft.fftfreq(n, 1.0 / n, device=DEV) for n in shape[:2])
    kz = torch.fft.rfftfreq(shape[2], 1.0 / shape[2], device=DEV)
    k = (kx[:, None, None] ** 2 + ky[None, :, None] ** 2 + kz[None, None, :] ** 2).sqrt()
    amp = torch.where((k >= 1) & (k <= min(shape) / 2), k.clamp(min=1) ** (-11.0 / 6.0), torch.zeros_like(k))
    out = torch.empty((nb,) + tuple(shape), device=DEV)
    for b0 in range(0, nb, 64):
        ph = torch.rand((min(64, nb - b0),) + tuple(k.shape), generator=gen, device=DEV) * (2 * math.pi)
        f = torch.fft.irfftn(torch.polar(amp.expand_as(ph), ph), s=tuple(shape), dim=(1, 2, 3))
        out[b0:b0 + 64] = (f - f.mean((1, 2, 3), keepdim=True)) / f.std((1, 2, 3), keepdim=True)
    return out


def _batch(case, seed):
    """A batch of micro-models as plain arrays. The lattice sizes and degrees
    are the case's; the seed gives the values (and the knots' jitter)."""
    g, sizes = (np.random.Generator(np.random.PCG64(k)) for k in (seed, 7))
    if "cells" in case:
        cells = _ints(case["cells"])
        nb = int(np.prod(cells))
        ncp = sizes.integers(max(case["ncp_lo"], case["degree"] + 1), max(case["ncp_hi"], case["degree"] + 1) + 1, (nb, 3))
        deg = np.full(nb, case["degree"])
        origin = np.stack(np.unravel_index(np.arange(nb), cells), 1).astype(float)
        jitter = case["knots"] == "jittered"
    else:
        nb = case["blocks"]
        ncp = sizes.choice(_ints(case["ncp"], ","), (nb, 3))
        deg = sizes.choice(_ints(case["degrees"], ","), nb)
        origin = g.uniform(0.0, 16.0, (nb, 3))
        jitter = case.get("knots") == "jittered"
    t, knots, koff, coff, total = _layout(ncp, deg, jitter, g)
    b = dict(ncp=ncp, deg=deg, t=t, knots=knots, koff=koff, coff=coff, total=total)
    if case.get("field") == "turbulence":
        P = _turbulence(nb, tuple(int(v) for v in ncp[0]), seed)  # one size for all: no gaps when it is a multiple of 64
        b["ctrl"] = torch.nn.functional.pad(P.reshape(nb, -1), (0, total // nb - P[0].numel())).reshape(-1)
    elif case["kind"] == "fit":
        b["ctrl"] = torch.zeros(total, device=DEV)
    elif case["kind"] == "search":
        b["ctrl"] = None
    else:
        b["ctrl"] = _sines(ncp, deg, t, coff, total, origin, g)
    return b


def _camera(case, seed):
    """Rays of a seeded camera that looks at the unit cube from distance 2:
    origins, unit directions, entry and exit (FP64)."""
    g = np.random.Generator(np.random.PCG64(seed + 1))
    w, h = case["width"], case["height"]
    v = g.normal(size=3)
    v /= np.linalg.norm(v)
    eye, fwd = 0.5 + 2.0 * v, -v
    right = np.cross(fwd, (0.0, 0.0, 1.0) if abs(fwd[2]) < 0.9 else (0.0, 1.0, 0.0))
    right /= np.linalg.norm(right)
    up = np.cross(right, fwd)
    th = math.tan(math.radians(13.9 if case["kind"] != "render" else 30.0) / 2)
    eye, fwd, right, up = (torch.tensor(a, device=DEV) for a in (eye, fwd, right, up))
    x = ((torch.arange(w, device=DEV, dtype=torch.float64) + 0.5) / w * 2 - 1) * th * max(1.0, w / h)
    y = (1 - (torch.arange(h, device=DEV, dtype=torch.float64) + 0.5) / h * 2) * th * max(1.0, h / w)
    d = (fwd + x[None, :, None] * right + y[:, None, None] * up).reshape(-1, 3)
    d = d / d.norm(dim=1, keepdim=True)
    a, b = (0.0 - eye) / d, (1.0 - eye) / d
    return eye.expand_as(d), d, torch.minimum(a, b).amax(1), torch.maximum(a, b).amin(1), g


def _positions(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed + 2)
    if case["kind"] == "rays":
        o, d, t0, t1, _ = _camera(case, seed)
        s = case["samples"]
        t1 = torch.maximum(t1, t0 + 0.05)
        jit = torch.rand(len(d), 1, generator=gen, device=DEV, dtype=torch.float64)
        t = t0[:, None] + (torch.arange(s, device=DEV)[None, :] + jit) / s * (t1 - t0)[:, None]
        out = torch.empty((len(d), s, 3), device=DEV)
        for a in range(3):
            out[:, :, a] = o[:, a, None] + d[:, a, None] * t
        return out.reshape(-1, 3)
    n = case["n"]
    if case["order"] == "scattered":
        return torch.rand(n, 3, generator=gen, device=DEV)
    lines = (n + 499) // 500  # 500 samples from one random point to another
    a, b = torch.rand(2, lines, 1, 3, generator=gen, device=DEV)
    s = (torch.arange(500, device=DEV)[None, :, None] + 0.5) / 500
    return (a + (b - a) * s).reshape(-1, 3)[:n].contiguous()


def _cells(case, seed):
    nb = int(np.prod(_ints(case["cells"])))
    m = np.arange(nb, dtype=np.int32)
    m[np.random.Generator(np.random.PCG64(seed + 3)).uniform(size=nb) < case["empty"]] = -1
    return torch.tensor(m, device=DEV)


def _transfer(g, n=256):
    x = np.linspace(0.0, 1.0, n)
    mu, sd, h = g.uniform(0, 1, (4, 5, 1)), g.uniform(0.04, 0.2, (4, 5, 1)), g.uniform(0.2, 1.0, (4, 5, 1))
    f = (h * np.exp(-0.5 * ((x - mu) / sd) ** 2)).sum(1)
    f /= f.max(1, keepdims=True)
    f[3] *= 0.08 * (np.abs(x - 0.5) > 0.08)
    return torch.tensor(f.T.astype(np.float32), device=DEV).contiguous()


_LIGHT = (0.26726124, 0.53452248, 0.80178373)  # unit vector along (1, 2, 3)
_TF_RANGE = (-4.0, 4.0)


def _frame(case, seed):
    o, d, t0, t1, g = _camera(case, seed)
    hit = t1 > t0
    t0, t1 = torch.where(hit, t0, torch.zeros_like(t0)), torch.where(hit, t1, -torch.ones_like(t1))
    return torch.cat([o, d, t0[:, None], t1[:, None]], 1).float().contiguous(), _transfer(g)


def _samples(case, seed):
    return _turbulence(case["blocks"], _ints(case["res"]), seed + 4)


def _cotangent(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed + 5)
    return torch.randn([case["blocks"], 4] + _ints(case["res"]), generator=gen, device=DEV)


# ------------------------------------------------------------ prepare, run

_MASK = dict(all=ALL, value=VALUE, gradient=GRAD, records=ALL | fa.OUT_INTERLEAVED)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, kind=kind)
    if kind == "search":
        return s | dict(y=_samples(case, seed))
    b = _batch(case, seed)
    m = fa.MicroModels(b["ncp"], np.repeat(b["deg"][:, None], 3, 1), b["koff"], b["coff"], b["knots"], b["ctrl"], DEV)
    s["models"] = m
    if "res" in case:
        s["res"] = tuple(_ints(case["res"]))
    if kind == "decode":
        m.lattice(case["dtype"])
        s["mask"] = _MASK[case["out"]]
        s["plan"] = fa.Plan(m, s["res"]) if case["how"] == "plan" else None
        s["tune"] = fa.FATune(0, 0, 0, 1, 0, 0) if case["how"] == "matrix" else None
    elif kind in ("query", "rays", "render"):
        m.lattice(case["dtype"])
        s["cells"] = _cells(case, seed)
        s["nb"] = tuple(_ints(case["cells"]))
        if kind == "render":
            s["rays"], s["tf"] = _frame(case, seed)
        else:
            s["xyz"] = _positions(case, seed)
    elif kind == "fitstep":
        s["ctrl"] = b["ctrl"].clone().requires_grad_()
        s["y"] = _samples(case, seed)
    elif kind == "grad4":
        s["ctrl"] = b["ctrl"].clone().requires_grad_()
        s["g"] = _cotangent(case, seed)
    elif kind == "fit":
        s["y"] = _samples(case, seed)
    return s


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "decode":
        return fa.decode(s["models"], s["res"], s["mask"], case["dtype"], plan=s["plan"], tune=s["tune"])
    if kind == "query":
        return fa.query(s["models"], s["xyz"], s["nb"], (0, 0, 0), (1, 1, 1), s["cells"], dtype=case["dtype"])
    if kind == "rays":
        return fa.query_rays(s["models"], s["xyz"], case["width"], case["height"], case["samples"], s["nb"],
                             (0, 0, 0), (1, 1, 1), s["cells"], dtype=case["dtype"])
    if kind == "render":
        return fa.render(s["models"], s["rays"], case["width"], case["height"], s["tf"], s["nb"], (0, 0, 0), (1, 1, 1),
                         s["cells"], case["samples"], opacity_max=case["opacity"], tf_range=_TF_RANGE, light=_LIGHT,
                         dtype=case["dtype"])
    if kind == "fitstep":
        s["ctrl"].grad = None
        loss = fa.FAFitMSE.apply(s["ctrl"], s["models"], s["res"], s["y"], None)
        loss.backward()
        return dict(loss=loss.detach(), grad=s["ctrl"].grad)
    if kind == "grad4":
        s["ctrl"].grad = None
        out = fa.FADecode.apply(s["ctrl"], s["models"], s["res"], ALL, None)
        out.backward(s["g"])
        return dict(out=out.detach(), grad=s["ctrl"].grad)
    if kind == "fit":
        return fa.fit(s["models"], s["res"], s["y"]).ctrl
    return fa.ncp_search(s["y"], case["degree"], case["lo"], case["hi"])


def work(case):
    """Inputs once, outputs once; FP operations of the contractions that a
    local tensor-product evaluation needs (2 per multiply-add)."""
    kind = case["kind"]
    if "cells" in case:
        p1 = case["degree"] + 1
        per = 2 * (2 * p1 ** 3 + 3 * p1 ** 2 + 4 * p1)  # z, y and x stage of one window, value and gradient
        cells = int(np.prod(_ints(case["cells"])))
        lattice = cells * ((case["ncp_lo"] + case["ncp_hi"]) / 2) ** 3 * (4 if case["dtype"] == "f32" else 2)
        if kind == "render":
            px = case["width"] * case["height"]
            # the samples that a frame takes depend on the data: a quarter of all as a figure
            return dict(bytes=px * 48 + lattice, flops=px * case["samples"] * per / 4)
        n = case["n"] if kind == "query" else case["width"] * case["height"] * case["samples"]
        return dict(bytes=n * 28 + min(lattice, n * p1 ** 3 * 4), flops=n * per)
    vox = case["blocks"] * int(np.prod(_ints(case["res"])))
    rx, ry, rz = _ints(case["res"])
    if kind == "search":
        ns = range(case["lo"], case["hi"] + 1)
        # per size: three contractions of the fit and a value decode; the samples are read once
        fl = sum(2 * case["blocks"] * (n * rx * ry * rz + n * n * rx * ry + n ** 3 * rx) + vox * 2 * 4 for n in ns)
        return dict(bytes=vox * 4 + case["blocks"] * len(ns) * 8, flops=fl)
    n = float(np.mean(_ints(case["ncp"], ",")))
    lattice = case["blocks"] * n ** 3
    if kind == "fit":
        return dict(bytes=vox * 4 + lattice * 4, flops=2 * case["blocks"] * (n * rx * ry * rz + n * n * rx * ry + n ** 3 * rx))
    p1 = 4
    if kind == "fitstep":  # samples and lattice in, gradient out, the loss; forward and transposed x, y, z stages
        return dict(bytes=vox * 4 + lattice * 8, flops=2 * 2 * (vox * p1 + case["blocks"] * n * ry * rz * 2 * p1))
    if kind == "grad4":  # four channels out, four cotangent channels in
        return dict(bytes=vox * 32 + lattice * 8, flops=2 * 2 * (vox * 4 * p1 + case["blocks"] * n * ry * rz * 5 * p1))
    ch = dict(all=4, records=4, gradient=3, value=1)[case["out"]]
    return dict(bytes=vox * 4 * ch + lattice * (4 if case["dtype"] == "f32" else 2),
                flops=2 * (vox * ch * p1 + case["blocks"] * n * ry * rz * 5 * p1))


# ------------------------------------------------- 64 bits, with torch alone

def _basis(t, n, p, u):
    """Dense N[i][j], N'[i][j] of the clamped basis of n functions at u."""
    t, u = np.asarray(t[:n + p + 1], np.float64), np.asarray(u, np.float64)
    s = np.clip(np.searchsorted(t, u, side="right") - 1, p, n - 1)
    N = np.zeros((len(u), n + p))
    N[np.arange(len(u)), s] = 1.0
    low = None
    for k in range(1, p + 1):
        low = N
        j = np.arange(n + p - k)
        a, b = t[j + k] - t[j], t[j + k + 1] - t[j + 1]
        a, b = np.where(a > 0, a, np.inf), np.where(b > 0, b, np.inf)
        N = (u[:, None] - t[j]) / a * low[:, j] + (t[j + k + 1] - u[:, None]) / b * low[:, j + 1]
    D = p * (low[:, :n] / a - low[:, 1:n + 1] / b)
    return torch.tensor(N[:, :n], device=DEV), torch.tensor(D, device=DEV)


def _grid(R):
    return np.arange(R, dtype=np.float32) / np.float32(R - 1)


def _axes(b, i, res, cache):
    """(N, D) of block i along x, y, z on its grid."""
    out = []
    for a in range(3):
        n, p = int(b["ncp"][i, a]), int(b["deg"][i])
        t = b["t"][i, a, :n + p + 1]
        key = (t.tobytes(), p, res[a])
        if key not in cache:
            cache[key] = _basis(t, n, p, _grid(res[a]))
        out.append(cache[key])
    return out


def _along(T, M, a):
    """Axis a of T contracted with the second index of M."""
    return torch.movedim(torch.tensordot(T, M, dims=([a], [1])), -1, a)


def _lattice(b, i, flat):
    n = b["ncp"][i]
    return flat[b["coff"][i]:b["coff"][i] + int(n.prod())].reshape(*map(int, n)).double()


def _stored(b, case):
    """The lattice values that the 2-byte storage holds, in 64 bits."""
    if case["dtype"] == "f32":
        return b["ctrl"]
    kind = torch.bfloat16 if case["dtype"] == "bf16" else torch.float16
    out = torch.zeros(b["total"], device=DEV, dtype=torch.float64)
    for i in range(len(b["ncp"])):
        c0, c1 = b["coff"][i], b["coff"][i] + int(b["ncp"][i].prod())
        P = b["ctrl"][c0:c1]
        s = P.abs().max()
        s = s if s > 0 else torch.ones_like(s)
        out[c0:c1] = (P * (1 / s)).clamp(-1, 1).to(kind).double() * s.double()
    return out


def _decode(b, flat, res, mask):
    chans = [c for c in range(4) if mask >> c & 1]
    out = torch.empty([len(b["ncp"]), len(chans)] + list(res), device=DEV, dtype=torch.float64)
    cache = {}
    for i in range(len(b["ncp"])):
        ax, P = _axes(b, i, res, cache), _lattice(b, i, flat)
        for k, c in enumerate(chans):
            f = P
            for a in (2, 1, 0):
                f = _along(f, ax[a][1 if c == a + 1 else 0], a)
            out[i, k] = f
    return out


def _adjoint(b, g, res, mask):
    chans = [c for c in range(4) if mask >> c & 1]
    out = torch.zeros(b["total"], device=DEV, dtype=torch.float64)
    cache = {}
    for i in range(len(b["ncp"])):
        ax, G = _axes(b, i, res, cache), 0.0
        for k, c in enumerate(chans):
            f = g[i, k].double()
            for a in range(3):
                f = _along(f, ax[a][1 if c == a + 1 else 0].T, a)
            G = G + f
        out[b["coff"][i]:b["coff"][i] + G.numel()] = G.reshape(-1)
    return out


def _at(b, flat, blk, u):
    """Value and d/du of micro-model blk[i] at block coordinates u[i] (one
    degree for the batch): span by counting, the triangular recursion, the
    (p+1)^3 window."""
    p = int(b["deg"][0])
    ncp = torch.tensor(b["ncp"], device=DEV)[blk]
    N, D, first = [], [], []
    for a in range(3):
        t = torch.tensor(b["t"][:, a].astype(np.float64), device=DEV)
        K = t.shape[1]
        inner = torch.where((torch.arange(K, device=DEV)[None, :] > p)
                            & (torch.arange(K, device=DEV)[None, :] < torch.tensor(b["ncp"][:, a:a + 1], device=DEV)),
                            t, torch.full_like(t, 9.0))
        x = u[:, a].double()
        s = torch.full_like(blk, p)
        for j in range(p + 1, K):
            s += x >= inner[blk, j]
        knot = lambda q: t.reshape(-1)[blk * K + s + q]  # noqa: E731
        left, right = [None] + [x - knot(1 - k) for k in range(1, p + 1)], [None] + [knot(k) - x for k in range(1, p + 1)]
        B = [torch.ones_like(x)]
        for k in range(1, p + 1):
            low, saved, new = B, 0.0, []
            for r in range(k):
                q = B[r] / (right[r + 1] + left[k - r])
                new.append(saved + right[r + 1] * q)
                saved = left[k - r] * q
            B = new + [saved]
        inv = [None] + [1.0 / (right[r] + left[p + 1 - r]) for r in range(1, p + 1)]
        dB = []
        for r in range(p + 1):
            d = low[r - 1] * inv[r] if r else torch.zeros_like(x)
            dB.append(p * (d - low[r] * inv[r + 1] if r < p else d))
        N.append(B)
        D.append(dB)
        first.append(s - p)
    base = torch.tensor(b["coff"], device=DEV)[blk] + (first[0] * ncp[:, 1] + first[1]) * ncp[:, 2] + first[2]
    out = torch.zeros((len(blk), 4), device=DEV, dtype=torch.float64)
    for i in range(p + 1):
        for j in range(p + 1):
            for k in range(p + 1):
                c = flat[base + (i * ncp[:, 1] + j) * ncp[:, 2] + k].double()
                out[:, 0] += N[0][i] * N[1][j] * N[2][k] * c
                out[:, 1] += D[0][i] * N[1][j] * N[2][k] * c
                out[:, 2] += N[0][i] * D[1][j] * N[2][k] * c
                out[:, 3] += N[0][i] * N[1][j] * D[2][k] * c
    return out


def _points(b, flat, case, cells, xyz):
    """_at() for positions in the unit cube; the cell and the block
    coordinate are FP32 numbers by definition. Zeros in empty cells."""
    out = torch.zeros((len(xyz), 4), device=DEV, dtype=torch.float64)
    nb = _ints(case["cells"])
    for q0 in range(0, len(xyz), 4_000_000):
        x = xyz[q0:q0 + 4_000_000]
        cell, u = torch.zeros(len(x), dtype=torch.long, device=DEV), torch.empty_like(x)
        for a in range(3):
            g = (x[:, a] * float(nb[a])).clamp(0.0, float(nb[a]))
            c = g.floor().clamp(max=float(nb[a] - 1))
            u[:, a] = g - c
            cell = cell * nb[a] + c.long()
        blk = cells[cell].long()
        r = _at(b, flat, blk.clamp(min=0), u) * torch.tensor([1.0] + [float(v) for v in nb], device=DEV, dtype=torch.float64)
        out[q0:q0 + 4_000_000] = torch.where((blk >= 0)[:, None], r, torch.zeros_like(r))
    return out


def _image(case, seed):
    """A frame whose rays run to their ends."""
    b = _batch(case, seed)
    flat, cells = _stored(b, case), _cells(case, seed)
    rays, tf = _frame(case, seed)
    S, n = case["samples"], tf.shape[0]
    tf, L = tf.double(), torch.tensor(_LIGHT, device=DEV, dtype=torch.float32).double()
    o, d, t0, t1 = rays[:, :3], rays[:, 3:6], rays[:, 6], rays[:, 7]
    dt, hit = (t1 - t0) / float(S), t1 > t0
    H = L - d.double()
    H = H / H.norm(dim=1, keepdim=True)
    C, A = torch.zeros((len(rays), 3), device=DEV, dtype=torch.float64), torch.zeros(len(rays), device=DEV, dtype=torch.float64)
    for s in range(S):
        t = t0 + (float(s) + 0.5) * dt
        e = _points(b, flat, case, cells, o + t[:, None] * d)
        q = ((e[:, 0] - _TF_RANGE[0]) / (_TF_RANGE[1] - _TF_RANGE[0]) * (n - 1)).clamp(0, n - 1)
        i = q.floor().clamp(max=n - 2).long()
        c = tf[i] + (q - i)[:, None] * (tf[i + 1] - tf[i])
        gl = e[:, 1:].norm(dim=1)
        N = e[:, 1:] / gl.clamp(min=1e-300)[:, None]
        lit = 0.3 + 0.6 * (N * L).sum(1).abs() + 0.3 * (N * H).sum(1).abs() ** 32.0
        w = torch.where(hit, (1 - A) * c[:, 3], torch.zeros_like(A))
        C += (w * torch.where(gl > 1e-6, lit, torch.full_like(lit, 0.3)))[:, None] * c[:, :3]
        A += w
    return torch.cat([C, A[:, None]], 1).reshape(case["height"], case["width"], 4)


def _pinv(t, n, p, R):
    return torch.linalg.pinv(_basis(t, n, p, _grid(R))[0].cpu()).to(DEV)


def exact(case, seed):
    kind = case["kind"]
    res = _ints(case["res"]) if "res" in case else None
    if kind == "render":
        # with early termination a ray near the threshold may stop a sample sooner or later
        if case["opacity"] < 1.0 or case["width"] * case["height"] * case["samples"] > 60_000_000:
            return None
        return _image(case, seed)
    if kind == "search":
        y = _samples(case, seed).double()
        out = torch.empty((case["blocks"], case["hi"] - case["lo"] + 1, 2), device=DEV, dtype=torch.float64)
        for n in range(case["lo"], case["hi"] + 1):
            p = case["degree"]
            t = np.clip((np.arange(n + p + 1) - p) / (n - p), 0.0, 1.0).astype(np.float32)
            f = y
            for a in range(3):
                f = _along(f, _basis(t, n, p, _grid(res[a]))[0] @ _pinv(t, n, p, res[a]), a + 1)
            r = (y - f).reshape(len(y), -1)
            out[:, n - case["lo"], 0] = r.abs().amax(1)
            out[:, n - case["lo"], 1] = r.square().mean(1).sqrt()
        return out
    b = _batch(case, seed)
    if kind == "decode":
        out = _decode(b, _stored(b, case), res, _MASK[case["out"]] & ALL)
        return out.movedim(1, -1) if case["out"] == "records" else out
    if kind in ("query", "rays"):
        return _points(b, _stored(b, case), case, _cells(case, seed), _positions(case, seed))
    if kind == "grad4":
        return dict(out=_decode(b, b["ctrl"], res, ALL), grad=_adjoint(b, _cotangent(case, seed), res, ALL))
    y = _samples(case, seed)
    if kind == "fitstep":
        r = _decode(b, b["ctrl"], res, VALUE) - y[:, None].double()
        return dict(loss=r.square().mean(), grad=_adjoint(b, r * (2.0 / r.numel()), res, VALUE))
    out, cache = torch.zeros(b["total"], device=DEV, dtype=torch.float64), {}
    for i in range(len(y)):
        f = y[i].double()
        for a in range(3):
            n, p = int(b["ncp"][i, a]), int(b["deg"][i])
            if (n, p, a) not in cache:
                cache[n, p, a] = _pinv(b["t"][i, a], n, p, res[a])
            f = _along(f, cache[n, p, a], a)
        out[b["coff"][i]:b["coff"][i] + f.numel()] = f.reshape(-1)
    return out
