"""Performance cases of the reconstruction library: the calls its users make, with their sizes.

A case is a dict of plain values: the operation, its precision, the scan and the sensor.
`prepare` makes what a program holds before the call (the model's device tables, the input and
output vectors), `run` makes one call through the public binding, `work` states the bytes and
operations of the mathematics, and `exact` gives the result in 64 bits from plain torch, built
from the equations alone (sub-element sum of the sensor, per-offset matrix products, LSQR,
FISTA).

The sizes are those of the repository's workloads: the 16 x 16 test scans, the 40 x 40
super-resolution pairs, the serving mix (sides 64 to 400, Nz 64 to 256, Nt = 4 Nz, K = 20
cones), the 200 x 200 and 400 x 400 vessel scans; the drawn cases fill the range between them,
ragged sizes included.
"""
from __future__ import annotations

import math

import torch

import paper_2009_10173_amd as aroam

SENSORS = {
    "4mm": dict(radius_m=4e-3, aperture_m=3e-3, hole_m=0.0, n_rings=20, f0_hz=50e6, frac_bw=1.0),
    "7mm": dict(radius_m=7e-3, aperture_m=2 * 7e-3 * 0.43, hole_m=0.9e-3, n_rings=17, f0_hz=50e6,
                frac_bw=1.0),
}
BAND = dict(f_lo_hz=0.5e6, f_hi_hz=80e6)
SPEED, RATE = 1500.0, 250e6  # m/s, samples/s


def _case(name, op, dtype, ny, nx, nz, nt, k, um=10, mode=1, sensor="4mm", **more):
    c = dict(op=op, dtype=dtype, ny=ny, nx=nx, nz=nz, nt=nt, k=k, um=um, mode=mode, sensor=sensor,
             taps=0, iters=0, sweeps=0, power=0)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest reconstruction: a few LSQR iterations of the 16 x 16 scan.  Launches and
        # latency are all of it.
        _case("lsqr fp32 16x16", "lsqr", "fp32", 16, 16, 32, 128, 4, mode=0, iters=8),
        # L1 reconstruction of the super-resolution pairs with the band-pass filtered model.
        _case("fista fp32 40x40 filtered", "fista", "fp32", 40, 40, 30, 128, 20, um=5, sensor="7mm",
              taps=16, iters=50, power=30),
        # Double precision, which every model carries, for checking: a small ragged scan ...
        _case("forward fp64 23x19", "forward", "fp64", 19, 23, 40, 200, 12),
        # ... and one of the serving mix.
        _case("adjoint fp64 96x96", "adjoint", "fp64", 96, 96, 64, 256, 20),
        # One apply of the smallest served scan.
        _case("forward fp32 64x64", "forward", "fp32", 64, 64, 64, 256, 20),
        # One apply of the 200 x 200 vessel scan.
        _case("adjoint fp32 200x200", "adjoint", "fp32", 200, 200, 128, 512, 20),
        # One apply of the 400 x 400 vessel scan, the largest workload.
        _case("forward fp32 400x400", "forward", "fp32", 400, 400, 256, 1024, 40, um=5),
        # A batch of three served scans of different sizes in one call, BF16.
        _case("batch forward bf16", "batch", "bf16", 128, 97, 64, 256, 20),
        # The reduced-precision applies of the 400 x 400 scan's refined reconstructions.
        _case("adjoint bf16 400x400", "adjoint", "bf16", 400, 400, 256, 1024, 40, um=5),
        _case("forward fp8 400x400", "forward", "fp8", 400, 400, 256, 1024, 40, um=5),
        # A served request as the scheduler runs it: BF16 iterations, FP32 refinement.
        _case("lsqr bf16 refined 96x96", "lsqr", "bf16", 96, 96, 64, 256, 20, sensor="7mm",
              iters=50, sweeps=2),
        # Band-pass filtering of the measured signals before a reconstruction.
        _case("filter fp32 200x200", "filter", "fp32", 200, 200, 128, 512, 20, taps=32),
    ]


def draw(rng):
    """One more case between the smallest and the largest of the listed ones."""
    def spread(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    op, dtype = rng.choice((("lsqr", "fp32"), ("fista", "fp32"), ("forward", "fp32"),
                            ("adjoint", "fp32"), ("forward", "fp64"), ("adjoint", "fp64"),
                            ("forward", "bf16"), ("adjoint", "bf16"), ("forward", "fp8"),
                            ("adjoint", "fp8"), ("batch", "bf16"), ("batch", "fp8"),
                            ("batch", "fp32"), ("filter", "fp32"), ("filter", "fp64")))
    solve = op in ("lsqr", "fista")
    top = {"fp64": 110, "fp32": 260, "bf16": 330, "fp8": 330}[dtype]
    ny, nx = spread(16, 110 if solve else top), spread(16, 110 if solve else top)
    nz = spread(24, 64 if solve or dtype == "fp64" else 160)
    nt = 4 * nz + rng.choice((0, 0, 0, rng.randrange(1, 40)))
    um = rng.choice((5, 10, 10))
    k = rng.randrange(4, 21) if um == 10 else rng.randrange(8, 33 if not solve else 21)
    c = _case("", op, dtype, ny, nx, nz, nt, k, um=um, mode=0 if k <= 6 else 1,
              sensor=rng.choice(("4mm", "7mm")))
    if op == "filter":
        c["taps"] = rng.randrange(8, 65)
    elif op == "lsqr":
        c["iters"] = rng.randrange(2, 6)
    elif op == "fista":
        c["iters"], c["power"], c["taps"] = rng.randrange(5, 21), 10, rng.choice((0, 16))
    return c


# --- inputs ------------------------------------------------------------------------------------

def _grid(c, ny=None, nx=None):
    return dict(c_mps=SPEED, fs_hz=RATE, nx=nx or c["nx"], ny=ny or c["ny"], step_m=c["um"] * 1e-6,
                nz=c["nz"], dz_m=c["um"] * 1e-6, nt=c["nt"], k_half=c["k"],
                footprint_mode=c["mode"])


def _filter(c):
    return dict(BAND, half_taps=c["taps"]) if c["taps"] else None


def _shapes(c):
    """(ny, nx) of every scan of the call: a batch holds three, of falling size."""
    if c["op"] != "batch":
        return [(c["ny"], c["nx"])]
    return [(max(1, c["ny"] * f // 4), max(1, c["nx"] * f // 4)) for f in (4, 3, 2)]


def _element(c):
    return torch.float64 if c["dtype"] == "fp64" else torch.float32


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _image(c, ny, nx, g):
    """Vessel-like tubes across the scan (axes quadratic in y, at all depths) over a weak dense
    background, as an iterate of a reconstruction holds them: [ny][nx][nz]."""
    f = dict(device="cuda", dtype=torch.float32)
    nz, x = c["nz"], 0.01 * torch.randn(ny, nx, c["nz"], generator=g, device="cuda")
    px, pz = torch.arange(nx, **f).view(1, nx, 1), torch.arange(nz, **f).view(1, 1, nz)
    t = torch.linspace(-1, 1, ny, **f).view(ny, 1, 1)
    n = max(2, min(12, ny * nx // 2000))
    r = torch.rand(n, 8, generator=g, device="cuda")
    for i in range(n):
        cx = nx * (r[i, 0] + 0.4 * (r[i, 1] - 0.5) * t + 0.3 * (r[i, 2] - 0.5) * t * t)
        cz = nz * (r[i, 3] + 0.4 * (r[i, 4] - 0.5) * t + 0.3 * (r[i, 5] - 0.5) * t * t)
        rad = (0.5 + 2.0 * r[i, 6]) * 10.0 / c["um"]
        x += (0.3 + 0.7 * r[i, 7]) * ((px - cx) ** 2 + (pz - cz) ** 2 <= rad * rad)
    return x.to(_element(c))


def _signals(c, ny, nx, g):
    """Pulses of point absorbers (arrival times hyperbolic in the scan position, EIR-shaped)
    with white noise at 20 dB below the peak, as a measurement holds them: [ny][nx][nt]."""
    f = dict(device="cuda", dtype=torch.float32)
    nt, s = c["nt"], 0.1 * torch.randn(ny, nx, c["nt"], generator=g, device="cuda")
    yy, xx = torch.arange(ny, **f).view(ny, 1, 1), torch.arange(nx, **f).view(1, nx, 1)
    n = torch.arange(nt, **f).view(1, 1, nt)
    count = max(2, min(10, ny * nx // 2000))
    r = torch.rand(count, 4, generator=g, device="cuda")
    sigma, omega = _eir(SENSORS[c["sensor"]])
    for i in range(count):
        rho2 = ((yy - ny * r[i, 0]) ** 2 + (xx - nx * r[i, 1]) ** 2)
        t = n - nt * (0.25 + 0.5 * r[i, 2]) - 0.02 * rho2
        a = (0.3 + 0.7 * r[i, 3]) * torch.exp(-rho2 / 400.0)
        s += a * torch.exp(-t * t / (2 * sigma * sigma)) * torch.sin(omega * t)
    return s.to(_element(c))


def _inputs(c, seed):
    g = _generator(seed)
    make = _image if c["op"] in ("forward", "batch") else _signals
    return [make(c, ny, nx, g) for ny, nx in _shapes(c)]


class _Models(list):
    """The models of a state, released with it."""

    def __del__(self):
        for m in self:
            m.close()


def prepare(case, seed):
    c = case
    low = c["dtype"] if c["dtype"] in ("bf16", "fp8") else None
    models = _Models(aroam.Model(SENSORS[c["sensor"]], _grid(c, ny, nx), filter=_filter(c),
                                 dtypes=("fp64", "fp32") + ((low,) if low else ()))
                     for ny, nx in _shapes(c))
    last = c["nz"] if c["op"] in ("adjoint", "lsqr", "fista") else c["nt"]
    outs = [torch.empty(ny, nx, last, dtype=_element(c), device="cuda") for ny, nx in _shapes(c)]
    return dict(case=c, models=models, ins=_inputs(c, seed), outs=outs)


def run(state):
    c, models, ins, outs = state["case"], state["models"], state["ins"], state["outs"]
    m, v, out, op = models[0], ins[0], outs[0], c["op"]
    if op == "forward":
        return m.forward(v, c["dtype"], out=out)
    if op == "adjoint":
        return m.adjoint(v, c["dtype"], out=out)
    if op == "filter":
        return m.filter_signals(v, out=out)
    if op == "batch":
        aroam.aroam_forward_batch([x.handle for x in models], aroam.DTYPES[c["dtype"]], ins, outs)
        return outs
    if op == "lsqr":
        return m.solve_lsqr(v, iters=c["iters"], inner=c["dtype"], outer="fp32",
                            refine_sweeps=c["sweeps"], out=out)[0]
    return m.solve_l1(v, iters=c["iters"], power_iters=c["power"], inner=c["dtype"], out=out)[0]


# --- the mathematics in 64 bits ------------------------------------------------------------------

def _eir(sensor):
    """Envelope width (samples) and carrier (rad per sample) of the impulse response."""
    band = sensor["f0_hz"] * sensor["frac_bw"] / (2 * math.sqrt(2 * math.log(2.0)))
    return RATE / (2 * math.pi * band), 2 * math.pi * sensor["f0_hz"] / RATE


def _elements(sensor):
    """Centres [M][3] (mm) and areas [M] of the cap's equal-angle rings of patches."""
    R = sensor["radius_m"] * 1e3
    rim = math.asin(sensor["aperture_m"] / (2 * sensor["radius_m"]))
    hole = math.asin(sensor["hole_m"] / (2 * sensor["radius_m"]))
    step = (rim - hole) / sensor["n_rings"]
    pos, area = [], []
    for ring in range(sensor["n_rings"]):
        a, b = hole + ring * step, hole + (ring + 1) * step
        mid = 0.5 * (a + b)
        n = 8 * max(1, int(math.floor(2 * math.pi * math.sin(mid) / (8 * step) + 0.5)))
        for i in range(n):
            phi = 2 * math.pi * (i + 0.5) / n
            pos.append((R * math.sin(mid) * math.cos(phi), R * math.sin(mid) * math.sin(phi),
                        -R * math.cos(mid)))
            area.append(2 * math.pi * R * R * (math.cos(a) - math.cos(b)) / n)
    return pos, area, rim


class _Table:
    """Columns of the model, one per class of offsets under the square's symmetry."""

    def __init__(self, c, values=True):
        self.c, sensor = c, SENSORS[c["sensor"]]
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        f = dict(device=dev, dtype=torch.float64)
        pos, area, rim = _elements(sensor)
        pos, area = torch.tensor(pos, **f), torch.tensor(area, **f)
        sigma, omega = _eir(sensor)
        K, nz, nt, mm = c["k"], c["nz"], c["nt"], c["um"] * 1e-3
        z = (torch.arange(nz, **f) - nz // 2) * mm
        rho = 2 * 0.71 * (SPEED / sensor["f0_hz"]) * 1e3 / math.sin(rim) + z.abs() * math.tan(rim)
        classes = [(a, b) for a in range(K + 1) for b in range(a + 1)]
        index = {ab: i for i, ab in enumerate(classes)}
        self.of = [[index[(max(abs(dy), abs(dx)), min(abs(dy), abs(dx)))]
                    for dx in range(-K, K + 1)] for dy in range(-K, K + 1)]
        lo = torch.full((len(classes), nz), nt, device=dev, dtype=torch.int64)
        hi = torch.full_like(lo, -1)
        H = torch.zeros(len(classes), nz, nt, **f) if values else None
        reach = 5.0 * sigma
        for i, (a, b) in enumerate(classes):
            p = torch.stack((torch.full_like(z, b * mm), torch.full_like(z, a * mm), z), 1)
            r = (p[:, None, :] - pos[None]).square().sum(2).sqrt()
            delay = (r - sensor["radius_m"] * 1e3) * (RATE / (SPEED * 1e3))
            l = (nt // 2 + delay.amin(1) - reach).ceil().long().clamp(min=0)
            h = (nt // 2 + delay.amax(1) + reach).floor().long().clamp(max=nt - 1)
            keep = h >= l
            if c["mode"] == 1:
                keep &= float(a * a + b * b) * mm * mm <= rho * rho
            lo[i], hi[i] = torch.where(keep, l, nt), torch.where(keep, h, -1)
            if not values or not bool(keep.any()):
                continue
            n = l[:, None] + torch.arange(int((h - l)[keep].max()) + 1, device=dev)  # [nz][w]
            weight = area / (2 * math.pi * r)
            out = torch.zeros(n.shape, **f)
            for k0 in range(0, nz, 64):
                tau = (n[k0:k0 + 64, :, None] - nt // 2) - delay[k0:k0 + 64, None, :]
                e = -torch.exp(-tau * tau / (2 * sigma * sigma)) * (
                    tau / (sigma * sigma) * torch.cos(omega * tau) + omega * torch.sin(omega * tau))
                e[tau.abs() > reach] = 0.0
                out[k0:k0 + 64] = (e * weight[k0:k0 + 64, None, :]).sum(2)
            inside = keep[:, None] & (n <= h[:, None])
            at = torch.arange(nz, device=dev)[:, None].expand_as(n)[inside]
            H[i, at, n[inside]] = out[inside]
        if c["taps"]:
            if values:
                H = _fir(H, c)
            on = hi >= 0
            lo = torch.where(on, (lo - c["taps"]).clamp(min=0), lo)
            hi = torch.where(on, (hi + c["taps"]).clamp(max=nt - 1), hi)
        self.H, self.lo, self.hi, self.blocks = H, lo, hi, []
        for k0 in range(0, nz, 32):  # depth blocks and the samples that their columns reach
            k1 = min(nz, k0 + 32)
            n0, n1 = int(lo[:, k0:k1].min()), int(hi[:, k0:k1].max()) + 1
            if n1 > n0:
                self.blocks.append((k0, k1, n0, n1))

    def entries(self):
        return (self.hi - self.lo + 1).clamp(min=0).sum(1).tolist()

    def apply(self, v, adjoint):
        """A v or A^T v for v [ny][nx][nz or nt]: one matrix product per row offset, depth block
        and group of scan rows, over all column offsets at once."""
        c, (ny, nx, _) = self.c, v.shape
        K, W = c["k"], 2 * c["k"] + 1
        out = torch.zeros(ny, nx, c["nz"] if adjoint else c["nt"], dtype=torch.float64,
                          device=v.device)
        pad = torch.nn.functional.pad(v, (0, 0, K, K, K, K))  # [ny + 2K][nx + 2K][L]
        for dy in range(-K, K + 1):
            of = torch.tensor(self.of[dy + K], device=v.device)
            for k0, k1, n0, n1 in self.blocks:
                T = self.H[of, k0:k1, n0:n1]  # [dx][k][n]
                if not bool((T != 0).any()):
                    continue
                i0, i1, o0, o1 = (n0, n1, k0, k1) if adjoint else (k0, k1, n0, n1)
                # classes do not depend on the sign of an offset: dx runs the same way for both
                T = (T.transpose(1, 2) if adjoint else T).reshape(W * (i1 - i0), o1 - o0)
                rows = max(1, int(2.5e8 / (nx * W * (i1 - i0))))
                for y0 in range(0, ny, rows):
                    y1 = min(ny, y0 + rows)
                    p = pad[y0 + K + dy:y1 + K + dy, :, i0:i1]
                    p = p.unfold(1, W, 1).permute(0, 1, 3, 2).reshape((y1 - y0) * nx, -1)
                    out[y0:y1, :, o0:o1] += (p @ T).view(y1 - y0, nx, o1 - o0)
        return out


def _fir(v, c):
    """The band-pass along the last axis: windowed sinc of 2 taps + 1 entries, zero outside."""
    L = c["taps"]
    d = torch.arange(-L, L + 1, dtype=torch.float64, device=v.device)
    lo, hi = 2 * BAND["f_lo_hz"] / RATE, 2 * BAND["f_hi_hz"] / RATE
    h = hi * torch.sinc(hi * d) - lo * torch.sinc(lo * d)
    h = h * (0.42 + 0.5 * torch.cos(math.pi * d / L) + 0.08 * torch.cos(2 * math.pi * d / L))
    p, n = torch.nn.functional.pad(v, (L, L)), v.shape[-1]
    out = torch.zeros_like(v)
    for j in range(2 * L + 1):
        out += h[j] * p[..., j:j + n]
    return out


def _lsqr(A, At, b1, b2, damp, gamma, iters, rule=False):
    """LSQR of min |b1 - A x|^2 + |b2 - gamma x|^2 + damp^2 |x|^2 from x = 0; with `rule`,
    damp^2 = 1e-2 |A^T b1|."""
    def norm(u, w):
        return math.sqrt(float(u.square().sum()) + (float(w.square().sum()) if w is not None else 0.0))

    def back(u, w):
        return At(u) + (gamma * w if w is not None else 0.0)

    beta = norm(b1, b2)
    u, w2 = b1 / beta, None if b2 is None else b2 / beta
    v = back(u, w2)
    alpha = norm(v, None)
    v = v / alpha
    lam = damp * damp
    if rule:
        lam = 1e-2 * alpha * beta
        damp = math.sqrt(lam)
    w, x, phibar, rhobar = v.clone(), torch.zeros_like(v), beta, alpha
    for _ in range(iters):
        u = A(v) - alpha * u
        w2 = None if w2 is None else gamma * v - alpha * w2
        beta = norm(u, w2)
        u, w2 = u / beta, None if w2 is None else w2 / beta
        v = back(u, w2) - beta * v
        alpha = norm(v, None)
        v = v / alpha
        rho1 = math.hypot(rhobar, damp)
        phibar = rhobar / rho1 * phibar
        rho = math.hypot(rho1, beta)
        cs, sn = rho1 / rho, beta / rho
        x = x + (cs * phibar / rho) * w
        w = v - (sn * alpha / rho) * w
        rhobar, phibar = -cs * alpha, sn * phibar
    return x, lam


def _fista(A, At, s, iters, power):
    v = torch.ones_like(At(s))
    v = v / v.norm()
    for _ in range(power):
        w = At(A(v))
        rq = float((v * w).sum())
        v = w / w.norm()
    L, lam = 2.02 * rq, 5e-3 * float(At(s).abs().max())
    x = torch.zeros_like(v)
    y, t = x, 1.0
    for _ in range(iters):
        p = y - 2.0 * At(A(y) - s) / L
        xn = p.sign() * (p.abs() - lam / L).clamp(min=0)
        tn = 0.5 * (1 + math.sqrt(1 + 4 * t * t))
        y, x, t = xn + (t - 1) / tn * (xn - x), xn, tn
    return x


def exact(case, seed):
    c, op = case, case["op"]
    ins = [v.double() for v in _inputs(c, seed)]
    if op == "filter":
        return _fir(ins[0], c)
    pairs = {"lsqr": (c["sweeps"] + 1) * (c["iters"] + 1), "fista": c["iters"] + c["power"]}.get(op, 1)
    if pairs * c["ny"] * c["nx"] * c["nz"] * (2 * c["k"] + 1) ** 2 > 4e11:
        return None  # too slow in this form
    table = _Table(c)

    def A(v):
        return table.apply(v, False)

    def At(v):
        return table.apply(v, True)

    if op == "forward":
        return A(ins[0])
    if op == "adjoint":
        return At(ins[0])
    if op == "batch":
        return [A(v) for v in ins]
    if op == "fista":
        return _fista(A, At, ins[0], c["iters"], c["power"])
    x, lam = _lsqr(A, At, ins[0], None, 0.0, 0.0, c["iters"], rule=True)
    for _ in range(c["sweeps"]):
        g = At(ins[0] - A(x)) - lam * x
        gam = math.sqrt(lam)
        x = x + _lsqr(A, At, torch.zeros_like(ins[0]), g / gam, 0.0, gam, c["iters"])[0]
    return x


def work(case):
    """Multiply-adds of the band entries over the scan positions that they reach, and every
    vector and table entry once."""
    c = case
    size = 8 if c["dtype"] == "fp64" else 4
    images = sum(ny * nx * c["nz"] for ny, nx in _shapes(c))
    signals = sum(ny * nx * c["nt"] for ny, nx in _shapes(c))
    if c["op"] == "filter":
        return dict(bytes=2.0 * signals * size, flops=2.0 * signals * (2 * c["taps"] + 1))
    t = _Table(c, values=False)
    n, K, macs = t.entries(), c["k"], 0.0
    for ny, nx in _shapes(c):
        for dy in range(-K, K + 1):
            for dx in range(-K, K + 1):
                macs += n[t.of[dy + K][dx + K]] * max(0, ny - abs(dy)) * max(0, nx - abs(dx))
    applies = {"lsqr": (c["sweeps"] + 1) * (2 * c["iters"] + 1) + 2 * c["sweeps"],
               "fista": 2 * (c["iters"] + c["power"]) + 1}.get(c["op"], 1)
    entry = {"fp64": 8, "fp32": 4, "bf16": 2, "fp8": 1}[c["dtype"]]
    return dict(bytes=float(images * size + signals * size + sum(n) * entry),
                flops=2.0 * macs * applies)
