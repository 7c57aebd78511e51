"""Performance cases of the non-uniform diffraction operators.

Each case is one call sequence that a user's program makes through the public
entry points (``Plan``, ``Batch``, the autograd functions, ``rs_direct``), at
sizes taken from the repository's own workloads and tests and at odd sizes
between them.  ``listed()`` names the cases, ``draw(rng)`` gives more of the
same ranges, ``prepare`` makes a case's inputs and handles on the GPU, ``run``
is one pass, ``work`` the bytes and operations a pass cannot do without, and
``exact`` the same outputs summed directly in float64.

The kinds of a case:

* ``oneshot``  new points every pass: ``set_points`` (type 3: both sets), then ``execute``
* ``execute``  points bound once, ``execute`` per pass
* ``adjoint``  points bound once, ``adjoint`` per pass
* ``train``    points bound once, forward and backward through the autograd function
* ``grid``     a uniform grid of its own pitch as the non-uniform plane, bound and executed
* ``batch``    many mixed planes one-shot in one ``Batch.run``
* ``rs``       Rayleigh-Sommerfeld direct summation
"""
import math
import random

import torch

import paper_1308_6644_amd as P

_BASE = dict(kind="oneshot", type=1, N=1024, M=1 << 20, points="clustered", lam=633e-9, g=4e-6, z=0.1,
             ox=0.0, oy=0.0, tf="asm", band="limited", tol=1e-6)


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a 64 x 64 plane from a few thousand points, range check included; latency and launches
        _case(name="t1_tiny", N=64, M=4096, points="uniform", lam=532e-9, g=8e-6, z=0.05, band="full"),
        # the paper's own experiment: a quadrant-sampled 256 x 256 source, Fresnel transfer function
        _case(name="t1_paper256", N=256, M=65536, points="quadrant", lam=500e-9, g=5e-6, z=0.008, tf="fresnel",
              band="full"),
        # a small phase-retrieval loop at display tolerance: forward and backward on points bound once, odd count
        _case(name="train_small", kind="train", type=2, N=256, M=30011, z=0.05, tol=1e-3),
        # the headline size, source side: 2^20 clustered points onto the N' = 2048 plane, range check deferred
        _case(name="t1_1m", ox=1e-3, defer=True),
        # the headline size, destination side, forward only
        _case(name="t2_1m", type=2, ox=1e-3, tf="fresnel", band="full", defer=True, forward_only=True),
        # reproducible results at the tightest tolerance, cropped plane, ragged count
        _case(name="t1_det_1e9", N=512, M=300007, points="uniform", z=0.02, tol=1e-9, deterministic=True, crop=True),
        # both planes non-uniform, ragged counts
        _case(name="t3_1m", type=3, M=1000003, M2=700001, defer=True),
        # hologram phase optimisation: forward and backward at 2^22 points in three clusters
        _case(name="cgh_4m", kind="train", type=2, N=2048, M=1 << 22, points="three_clusters", lam=532e-9, z=0.2),
        # the largest plane: 2^24 points with a dense region of interest, metres of propagation
        _case(name="t2_roi_16m", type=2, N=4096, M=1 << 24, points="roi", lam=532e-9, z=1.0, defer=True),
        # scaled diffraction: a 2x zoom onto a 2048 x 2048 grid
        _case(name="zoom_2048", kind="grid", type=2, nx=2048, ny=2048, pitch=2e-6),
        # many mixed planes at once
        _case(name="batch_16", kind="batch", planes=16, pick=4, max_n=1024, max_m=1000000),
        # the accuracy reference of the paper: every pair of 256 x 256 points
        _case(name="rs_65536", kind="rs", M=65536, M2=65536, points="quadrant", N=256, lam=500e-9, g=5e-6, z=0.008),
    ]


def _log_int(rng, lo, hi):
    return int(math.floor(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["oneshot"] * 5 + ["execute"] * 2 + ["adjoint"] * 2 + ["train"] * 2 + ["grid", "batch", "rs"])
    if kind == "rs":
        n = rng.choice([64, 128, 256])
        m1 = _log_int(rng, 1000, 65536)
        return _case(kind="rs", N=n, M=m1, M2=_log_int(rng, 1000, 65536), points=rng.choice(["uniform", "clustered"]),
                     lam=rng.choice([500e-9, 633e-9]), g=5e-6, z=rng.uniform(0.004, 0.2), ox=rng.uniform(0, 2e-4))
    if kind == "batch":
        return _case(kind="batch", planes=rng.randint(3, 16), pick=rng.randint(10, 100000),
                     max_n=rng.choice([256, 512, 1024]), max_m=_log_int(rng, 20000, 1000000))
    n = rng.choice([32, 64, 128, 256, 512, 1024, 2048])
    tf = rng.choice(["asm", "asm", "fresnel"])
    c = _case(kind=kind, N=n, type=rng.choice([1, 2, 3]), M=_log_int(rng, 1000, min(1 << 22, 64 * n * n)),
              points=rng.choice(["uniform", "clustered", "three_clusters"]),
              lam=rng.choice([500e-9, 532e-9, 633e-9]), g=rng.choice([4e-6, 5e-6, 8e-6]),
              z=math.exp(rng.uniform(math.log(0.005), math.log(1.0))), ox=rng.choice([0.0, rng.uniform(0, 0.3) * n * 4e-6]),
              tf=tf, band=rng.choice(["full", "limited", "limited"]) if tf == "asm" else "full",
              tol=rng.choice([1e-3, 1e-6, 1e-6, 1e-9]), defer=rng.random() < 0.5)
    if kind == "grid":
        s = rng.uniform(0.4, 1.0)
        c.update(type=rng.choice([1, 2]), nx=_log_int(rng, 30, 2 * n), ny=_log_int(rng, 30, 2 * n))
        c.update(pitch=s * c["g"] * n / max(c["nx"], c["ny"]) * 0.999, defer=False)
        return c
    if c["type"] == 3:
        c["M2"] = _log_int(rng, 1000, min(1 << 21, 64 * n * n))
        c["M"] = min(c["M"], 1 << 21)
    if kind in ("adjoint", "train") and c["type"] == 3:
        c["defer"] = False
    if kind in ("oneshot", "execute") and c["type"] == 2 and rng.random() < 0.4:
        c["forward_only"] = True
    if c["type"] == 1 and kind in ("oneshot", "execute") and rng.random() < 0.3:
        c["crop"] = True
    if n <= 1024 and c["M"] <= 500000 and rng.random() < 0.2:
        c["deterministic"] = True
    return c


# ------------------------------------------------------------------ inputs
def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((1000003 * (seed + 1) + 7919 * stream) % (1 << 62))
    return g


def _uniform(g, n, lo, hi):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo


def _gauss(g, n, centre, sigma, half):
    """Normal deviates truncated to [-half, half) (by the inverse distribution function)."""
    r = math.sqrt(2.0) * sigma
    lo, hi = math.erf((-half - centre) / r), math.erf((half - centre) / r)
    u = _uniform(g, n, lo, hi).clamp_(-1 + 1e-15, 1 - 1e-15)
    return (centre + r * torch.erfinv(u)).clamp_(-half, half * (1 - 1e-12))


def _points(kind, g, M, N, pitch):
    """M points (float64 metres) in the N pitch window, in shuffled order."""
    W = N * pitch
    h = W / 2
    if kind == "uniform":
        return _uniform(g, M, -h, h), _uniform(g, M, -h, h)
    if kind == "clustered":  # 70 % in a Gaussian of 0.1 W, the rest uniform
        m = int(round(0.7 * M))
        x = torch.cat([_gauss(g, m, 0.0, 0.1 * W, h), _uniform(g, M - m, -h, h)])
        y = torch.cat([_gauss(g, m, 0.0, 0.1 * W, h), _uniform(g, M - m, -h, h)])
    elif kind == "three_clusters":
        cs = _uniform(g, 6, -0.3 * W, 0.3 * W).tolist()
        ms = [M // 3, M // 3, M - 2 * (M // 3)]
        x = torch.cat([_gauss(g, ms[i], cs[2 * i], 0.05 * W, h) for i in range(3)])
        y = torch.cat([_gauss(g, ms[i], cs[2 * i + 1], 0.05 * W, h) for i in range(3)])
    elif kind == "quadrant":  # (N/2)^2 points per quadrant at 0.9 / 0.8 / 0.7 / 1.0 of the pitch
        a = (torch.arange(N // 2, device="cuda", dtype=torch.float64) + 0.5) * pitch
        xs, ys = [], []
        for sx, sy, f in ((1, 1, 0.9), (-1, 1, 0.8), (-1, -1, 0.7), (1, -1, 1.0)):
            gy, gx = torch.meshgrid(sy * f * a, sx * f * a, indexing="ij")
            xs.append(gx.reshape(-1))
            ys.append(gy.reshape(-1))
        x, y = torch.cat(xs), torch.cat(ys)
    elif kind == "roi":  # jittered pixels, four points per pixel in a central 512 x 512 region
        n_roi = 1024 * 1024
        q = torch.arange(1024, device="cuda", dtype=torch.float64) * 0.5 - 256
        ry, rx = torch.meshgrid(q, q, indexing="ij")
        bg = torch.randperm(N * N, generator=g, device="cuda")
        by, bx = bg // N - N // 2, bg % N - N // 2
        keep = ((bx < -256) | (bx >= 256) | (by < -256) | (by >= 256)).nonzero().reshape(-1)[:M - n_roi]
        j = [_uniform(g, k, 0.0, s) for k, s in ((keep.numel(), 1.0), (n_roi, 0.5)) for _ in range(2)]
        x = torch.cat([bx[keep].double() + j[0], rx.reshape(-1) + j[2]]) * pitch
        y = torch.cat([by[keep].double() + j[1], ry.reshape(-1) + j[3]]) * pitch
    else:
        raise ValueError(kind)
    p = torch.randperm(x.numel(), generator=g, device="cuda")
    return x[p].clamp(-h, h).contiguous(), y[p].clamp(-h, h).contiguous()


def _phase(g, shape):
    """Unit-amplitude values of random phase, complex64."""
    th = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) * (2 * math.pi)
    return torch.polar(torch.ones_like(th), th).to(torch.complex64)


def _point_counts(c):
    """(points of the first set, of the second) as the generators make them."""
    n = (c["N"] // 2) ** 2 * 4 if c["points"] == "quadrant" else c["M"]
    return n, c.get("M2", 0)


def _inputs(c, seed):
    """The case's arrays: points, the operator's input, the cotangent of its output."""
    g = _generator(seed, 1)
    d = {}
    if c["kind"] == "grid":
        npts = c["nx"] * c["ny"]
    else:
        d["x"], d["y"] = _points(c["points"], g, c["M"], c["N"], c["g"])
        npts = d["x"].numel()
        if c["type"] == 3 or c["kind"] == "rs":
            k2 = "uniform" if c["kind"] == "rs" else c["points"]
            d["x2"], d["y2"] = _points(k2, g, c["M2"], c["N"], c["g"])
    n, np_ = c["N"], 2 * c["N"]
    if c["kind"] == "rs":
        d["v"] = _phase(g, (npts,)) * (c["g"] * c["g"])
        return d
    fwd_in = (n, n) if c["type"] == 2 else (npts,)
    fwd_out = {1: (np_, np_), 2: (npts,), 3: (c.get("M2", 0),)}[c["type"]]
    if c["kind"] != "adjoint":
        d["v"] = _phase(g, fwd_in)
    if c["kind"] in ("adjoint", "train"):
        d["w"] = _phase(g, fwd_out)
    return d


def _plane_specs(c):
    """The batch's planes, each a one-shot case of its own."""
    r = random.Random(c["pick"])
    ns = [n for n in (256, 512, 1024) if n <= c["max_n"]]
    out = []
    for _ in range(c["planes"]):
        tf = r.choice(["asm", "fresnel"])
        out.append(_case(N=r.choice(ns), M=_log_int(r, 10000, c["max_m"]), type=r.choice([1, 2]),
                         z=r.uniform(0.005, 0.5), tf=tf, band="limited" if tf == "asm" else "full"))
    return out


def _params(c):
    return dict(N=c["N"], type=c["type"], lam=c["lam"], z=c["z"], g=c["g"], tf=c["tf"], band=c["band"], ox=c["ox"],
                oy=c["oy"], tol=c["tol"], crop=c.get("crop", False), defer_range_check=c.get("defer", False),
                deterministic=c.get("deterministic", False), forward_only=c.get("forward_only", False))


def prepare(case, seed):
    if case["kind"] == "rs":
        return dict(case=case, **_inputs(case, seed))
    if case["kind"] == "batch":
        specs = _plane_specs(case)
        ds = [_inputs(s, seed * 64 + i) for i, s in enumerate(specs)]
        params = []
        for s in specs:
            p = _params(s)
            params.append({k: p[k] for k in ("N", "type", "lam", "z", "g", "tf", "band", "ox", "oy", "tol")})
        outs = [torch.empty((2 * s["N"], 2 * s["N"]) if s["type"] == 1 else (s["M"],), dtype=torch.complex64,
                            device="cuda") for s in specs]
        return dict(case=case, batch=P.Batch(params), xs=[d["x"] for d in ds], ys=[d["y"] for d in ds],
                    ins=[d["v"] for d in ds], outs=outs)
    st = dict(case=case, plan=P.Plan(**_params(case)), **_inputs(case, seed))
    if case["kind"] in ("execute", "adjoint", "train"):
        st["plan"].set_points(st["x"], st["y"])
        if case["type"] == 3:
            st["plan"].set_dest_points(st["x2"], st["y2"])
    if case["kind"] == "train":
        st["v"].requires_grad_(True)
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "batch":
        return st["batch"].run(st["xs"], st["ys"], st["ins"], st["outs"])
    if kind == "rs":
        return P.rs_direct(st["x"], st["y"], st["v"], st["x2"], st["y2"], lam=c["lam"], z=c["z"], ox=c["ox"],
                           oy=c["oy"])
    plan = st["plan"]
    if kind == "oneshot":
        plan.set_points(st["x"], st["y"])
        if c["type"] == 3:
            plan.set_dest_points(st["x2"], st["y2"])
        return plan.execute(st["v"])
    if kind == "grid":
        plan.set_grid_points(c["nx"], c["ny"], c["pitch"])
        return plan.execute(st["v"])
    if kind == "execute":
        return plan.execute(st["v"])
    if kind == "adjoint":
        return plan.adjoint(st["w"])
    op = {1: P.nuasm1, 2: P.nuasm2, 3: P.nuasm3}[c["type"]]
    u = op(st["v"], plan)
    (grad,) = torch.autograd.grad(u, st["v"], st["w"])
    return u.detach(), grad


# -------------------------------------------------------------------- work
def work(case):
    """Bytes: points (16 B), values and planes (8 B) read or written once per
    pass.  Operations: the two 2-D transforms of the N' x N' spectrum, a
    complex multiply-add per tap (w^2 a point, or w per axis on a grid), 40 a
    pair of the direct sum."""
    c = case
    if c["kind"] == "batch":
        ws = [work(s) for s in _plane_specs(c)]
        return {k: float(sum(w[k] for w in ws)) for k in ("bytes", "flops")}
    m1, m2 = _point_counts(c)
    if c["kind"] == "rs":
        return {"bytes": 24.0 * m1 + 24.0 * m2, "flops": 40.0 * m1 * m2}
    n, np_ = c["N"], 2 * c["N"]
    w = math.ceil(-math.log10(c["tol"]) - 1e-9) + 1
    bind = c["kind"] == "oneshot"
    if c["kind"] == "grid":
        m1 = c["nx"] * c["ny"]
    plane = n * n if c["type"] == 2 or c.get("crop") else np_ * np_
    pts = 8.0 * m1 + (16.0 * m1 if bind else 0.0)
    if c["type"] == 3:
        pts += 8.0 * m2 + (16.0 * m2 if bind else 0.0)
    io = pts + (8.0 * plane if c["type"] != 3 else 0.0)
    fft = 2 * 5.0 * np_ * np_ * 2 * math.log2(np_)
    taps = (m1 + (m2 if c["type"] == 3 else 0)) * (2.0 * w * 4 if c["kind"] == "grid" else w * w * 4.0)
    twice = 2 if c["kind"] == "train" else 1
    return {"bytes": twice * io, "flops": twice * (fft + taps)}


# ------------------------------------------------------- float64 direct sums
def _cis(cycles):
    a = 2 * math.pi * (cycles - torch.round(cycles))
    return torch.complex(torch.cos(a), torch.sin(a))


def _band(c, o, df):
    np_ = 2 * c["N"]
    lo, hi = -np_ // 2, np_ // 2 - 1
    if c["tf"] != "asm" or c["band"] != "limited":
        return lo, hi
    z, lam, s = c["z"], c["lam"], c["N"] * c["g"]

    def f(t):
        return t / (lam * math.sqrt(z * z + t * t))
    return max(lo, math.ceil(f(o - s) / df)), min(hi, math.floor(f(o + s) / df))


def _spectrum(c, conj):
    """(kx, ky, H on ky x kx) over the band, complex128."""
    np_, g, z, lam = 2 * c["N"], c["g"], c["z"], c["lam"]
    df = 1.0 / (np_ * g)
    ks = []
    for o in (c["ox"], c["oy"]):
        lo, hi = _band(c, o, df)
        ks.append(torch.arange(lo, hi + 1, device="cuda", dtype=torch.float64))
    kx, ky = ks
    zl = z / lam
    if c["tf"] == "fresnel":
        m = torch.arange(-np_ // 2, np_ // 2, device="cuda", dtype=torch.float64)
        ax = []
        for o in (c["ox"], c["oy"]):
            h = _cis((m * g + o) ** 2 / (2 * lam * z))
            ax.append(torch.fft.fftshift(torch.fft.fft(torch.fft.ifftshift(h))))
        amp = g * g / (1j * lam * z) * complex(math.cos(2 * math.pi * (zl % 1.0)), math.sin(2 * math.pi * (zl % 1.0)))
        h = amp * ax[1][:, None] * ax[0][None, :]
    else:
        t = (lam * df) ** 2 * (kx[None, :] ** 2 + ky[:, None] ** 2)
        s = torch.sqrt((1 - t).clamp(min=0))
        cyc = (zl - round(zl)) - zl * t / (1 + s) + df * (kx[None, :] * c["ox"] + ky[:, None] * c["oy"])
        h = _cis(cyc)
        h[t > 1] = 0
    return kx, ky, h.conj() if conj else h


def _to_spectrum(c, x, y, v, kx, ky):
    """sum_j v_j exp(-2 pi i df k . p_j) on ky x kx."""
    df = 1.0 / (2 * c["N"] * c["g"])
    out = torch.zeros(ky.numel(), kx.numel(), dtype=torch.complex128, device="cuda")
    for a in range(0, x.numel(), 16384):
        b = slice(a, a + 16384)
        ex = _cis(-df * x[b][:, None] * kx[None, :])
        ey = _cis(-df * ky[:, None] * y[b][None, :]) * v[b].to(torch.complex128)[None, :]
        out += ey @ ex
    return out


def _to_points(c, x, y, spec, kx, ky):
    """N'^-2 sum_k spec(k) exp(2 pi i df k . q_j)."""
    np_ = 2 * c["N"]
    df = 1.0 / (np_ * c["g"])
    out = torch.empty(x.numel(), dtype=torch.complex128, device="cuda")
    for a in range(0, x.numel(), 16384):
        b = slice(a, a + 16384)
        ey = _cis(df * y[b][:, None] * ky[None, :])
        ex = _cis(df * x[b][:, None] * kx[None, :])
        out[b] = ((ey @ spec) * ex).sum(1)
    return out / (np_ * np_)


def _plane_to_spectrum(c, u, kx, ky):
    np_, m = 2 * c["N"], u.shape[0]
    p = torch.zeros(np_, np_, dtype=torch.complex128, device="cuda")
    o = (np_ - m) // 2
    p[o:o + m, o:o + m] = u.to(torch.complex128)
    f = torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(p)))
    h = np_ // 2
    return f[int(ky[0]) + h:int(ky[-1]) + h + 1, int(kx[0]) + h:int(kx[-1]) + h + 1]


def _spectrum_to_plane(c, spec, kx, ky, crop):
    np_, h = 2 * c["N"], c["N"]
    f = torch.zeros(np_, np_, dtype=torch.complex128, device="cuda")
    f[int(ky[0]) + h:int(ky[-1]) + h + 1, int(kx[0]) + h:int(kx[-1]) + h + 1] = spec
    u = torch.fft.fftshift(torch.fft.ifft2(torch.fft.ifftshift(f)))
    return u[h // 2:h // 2 + h, h // 2:h // 2 + h] if crop else u


def _direct(c, d, adjoint):
    v = d["w"] if adjoint else d["v"].detach()
    kx, ky, h = _spectrum(c, adjoint)
    if kx.numel() == 0 or ky.numel() == 0:
        return None
    if c["kind"] == "grid":
        xs = (torch.arange(c["nx"], device="cuda", dtype=torch.float64) - c["nx"] // 2) * c["pitch"]
        ys = (torch.arange(c["ny"], device="cuda", dtype=torch.float64) - c["ny"] // 2) * c["pitch"]
        np_ = 2 * c["N"]
        df = 1.0 / (np_ * c["g"])
        ex, ey = _cis(df * xs[:, None] * kx[None, :]), _cis(df * ys[:, None] * ky[None, :])
        if c["type"] == 2:
            s = _plane_to_spectrum(c, v, kx, ky) * h
            return ((ey @ s) @ ex.transpose(0, 1).contiguous()).reshape(-1) / (np_ * np_)
        s = (ey.conj().transpose(0, 1).contiguous() @ v.reshape(c["ny"], c["nx"]).to(torch.complex128)) @ ex.conj()
        return _spectrum_to_plane(c, s * h, kx, ky, c.get("crop", False))
    if c["type"] == 3:
        src, dst = (("x2", "y2"), ("x", "y")) if adjoint else (("x", "y"), ("x2", "y2"))
        s = _to_spectrum(c, d[src[0]], d[src[1]], v, kx, ky) * h
        return _to_points(c, d[dst[0]], d[dst[1]], s, kx, ky)
    if (c["type"] == 1) != adjoint:
        s = _to_spectrum(c, d["x"], d["y"], v, kx, ky) * h
        return _spectrum_to_plane(c, s, kx, ky, c["type"] == 2 or c.get("crop", False))
    return _to_points(c, d["x"], d["y"], _plane_to_spectrum(c, v, kx, ky) * h, kx, ky)


def _direct_rs(c, d):
    z, lam = c["z"], c["lam"]
    out = torch.empty(d["x2"].numel(), dtype=torch.complex128, device="cuda")
    v = d["v"].to(torch.complex128)
    k = 2 * math.pi / lam
    for a in range(0, out.numel(), 1024):
        b = slice(a, a + 1024)
        rho2 = (d["x2"][b][:, None] + c["ox"] - d["x"][None, :]) ** 2 + (d["y2"][b][:, None] + c["oy"] - d["y"][None, :]) ** 2
        r = torch.sqrt(rho2 + z * z)
        zl = abs(z) / lam
        t = _cis((zl - round(zl)) + rho2 / (lam * (r + abs(z)))) * torch.complex(z / r ** 3, -k * z / (r * r))
        out[b] = t @ v / (2 * math.pi)
    return out


def _direct_cost(c):
    """Operations of the direct sums, in complex128 products of matrices."""
    if c["kind"] in ("grid", "rs"):
        return 0.0
    df = 1.0 / (2 * c["N"] * c["g"])
    k = [max(0, hi - lo + 1) for lo, hi in (_band(c, c["ox"], df), _band(c, c["oy"], df))]
    m = sum(_point_counts(c))
    return 8.0 * m * k[0] * k[1] * (2 if c["kind"] == "train" else 1)


def exact(case, seed):
    if case["kind"] == "batch":
        specs = _plane_specs(case)
        if sum(_direct_cost(s) for s in specs) > 6e14:
            return None
        return [_direct(s, _inputs(s, seed * 64 + i), False) for i, s in enumerate(specs)]
    if _direct_cost(case) > 6e14:
        return None
    d = _inputs(case, seed)
    if case["kind"] == "rs":
        return _direct_rs(case, d)
    if case["kind"] == "train":
        return _direct(case, d, False), _direct(case, d, True)
    return _direct(case, d, case["kind"] == "adjoint")
