"""The work that users of this library have it do, as cases that can be timed.

A case names an entry point and the sizes of its work unit(s).  Shapes are
those of the repository's workload recipes (the 256-template smoke case, the
2-detector work unit of 2000 sky points, the uneven and the 32-spindown
batches, the semi-coherent segments) at full size or scaled down, and a few
generic ones between them: a follow-up of one sky point, small calls on the
static scratch, a frequency grid finer than the SFT bins.

Inputs are drawn on the device from the seed alone: SFTs of unit-variance
complex Gaussian noise with a few signals of SNR 8 to 20 added, time stamps
with gaps or jitter over the observation, detectors on a rotating Earth in
circular orbit, antenna patterns of two sites.  2F is the F-statistic of
include/fstat.h, and `exact` evaluates that definition term by term in FP64.
"""
import math

import numpy as np
import torch

import paper_0904_1826_amd as P

DEV = "cuda"
T_SFT = 1800.0
EPOCH = 8.0e8
ORBIT_R, ORBIT_W, OBLIQUITY = 499.005, 2.0 * math.pi / (365.25636 * 86400.0), math.radians(23.4393)
EARTH_R, SIDEREAL_W = 0.02127, 2.0 * math.pi / 86164.0905
# latitude, longitude, azimuths of the two arms (radians)
SITES = tuple(tuple(math.radians(x) for x in s) for s in ((46.5, -119.4, 126.0, 216.0), (30.6, -90.8, 198.0, 288.0)))


def _unit(name, entry, n_sft, n_sky, n_fd, n_f, **more):
    """A case: `entry` is the entry point, the sizes are those of its work
    unit (of the largest of them, for `units` > 1).  step: frequency step in
    SFT bins; keep: fraction of the time slots that hold an SFT; fd_lo: the
    spindowns run from fd_lo to 0."""
    c = dict(entry=entry, n_det=2, n_sft=n_sft, n_sky=n_sky, n_fd=n_fd, n_f=n_f, dterms=8, f0=1000.0, step=1.0,
             keep=0.6, fd_lo=-1.0e-9, storage="c64", phase="fp64", kernel="auto", coef="f32", fafb=False, top_k=0,
             full=True, units=1)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one sky point, no spindown, 256 templates, a few dozen SFTs of one detector;
        # launches and waits are all there is
        _unit("smoke-256", "compute", 32, 1, 1, 256, n_det=1, dterms=16, f0=100.0, keep=1.0, fd_lo=0.0),
        # a serving loop that may not allocate: small units on the library's static scratch
        _unit("noalloc-small", "noalloc", 48, 12, 4, 700, n_det=1, f0=310.0, keep=1.0),
        # the step before the demodulation: positions, velocities and antenna patterns of a work unit
        _unit("detector-inputs", "detector", 2000, 2000, 1, 1),
        # follow-up of one sky point over many spindowns, with Fa and Fb for the amplitude parameters
        _unit("followup-one-sky", "compute", 1500, 1, 51, 1801, dterms=16, f0=612.5, fafb=True),
        # the work unit of a search: 2 detectors, 2000 SFTs, 2000 sky points x 8 spindowns x 2 Hz
        _unit("workunit", "compute", 2000, 2000, 8, 3600),
        # a search client's call: 16-bit SFTs, only the strongest candidates kept, ragged sizes
        _unit("bf16-toplist", "compute", 801, 301, 8, 2701, f0=431.0, storage="bf16", top_k=20, full=False),
        # a frequency grid finer than the SFT bins, split phase, half-precision SFTs
        _unit("fine-grid-split", "compute", 701, 61, 5, 3001, n_det=1, f0=187.25, step=0.37, storage="fp16",
              phase="split"),
        # the FP16-coefficient form
        _unit("coef16", "compute", 601, 200, 8, 3600, storage="bf16", coef="f16"),
        # the term-by-term kernel
        _unit("direct", "compute", 600, 60, 8, 3600, kernel="direct"),
        # several clients' work units in one call: uneven SFT counts, bands, sky grids and spindowns
        _unit("batch-uneven", "batch", 800, 500, 16, 3600, keep=1.0, units=10),
        # wide bands with 32 spindowns each, BF16 SFTs
        _unit("batch-wide-bf16", "batch", 2200, 40, 32, 14400, dterms=16, keep=1.0, storage="bf16", units=3),
        # the incoherent stage: 2F summed over time segments on one template grid
        _unit("semicoherent", "semicoherent", 100, 500, 8, 3600, units=6),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: an entry point, log-uniform sizes, an
    option or two; at most a sixth of the largest listed case's work."""
    entry = rng.choice(["compute", "compute", "compute", "compute", "noalloc", "batch", "semicoherent", "detector"])
    if entry == "detector":
        return _unit(None, entry, _log(rng, 60, 4000), _log(rng, 1, 4000), 1, 1, n_det=rng.choice([1, 2]))
    more = dict(n_det=rng.choice([1, 2]), dterms=rng.choice([8, 8, 16, 16, 12]), f0=round(rng.uniform(50.0, 1500.0), 3),
                keep=rng.choice([1.0, 0.6]), storage=rng.choice(["c64", "c64", "bf16", "fp16"]),
                phase=rng.choice(["fp64", "fp64", "fp64", "split"]))
    more["step"] = rng.choice([1.0, 1.0, 1.0, 0.5, round(rng.uniform(0.05, 0.95), 3)])
    n_sft, n_sky, n_fd, n_f = _log(rng, 30, 2000), _log(rng, 1, 2000), rng.randint(1, 40), _log(rng, 100, 7200)
    if rng.random() < 0.5:
        n_fd = rng.randint(4, 16)
    if entry == "noalloc":
        n_sft, n_sky, n_f = _log(rng, 30, 300), _log(rng, 1, 60), _log(rng, 100, 2000)
    elif entry == "batch":
        more.update(units=rng.randint(2, 12), step=1.0)
    elif entry == "semicoherent":
        more.update(units=rng.randint(2, 8))
        n_sft = _log(rng, 30, 300)
    else:
        more.update(rng.choice([{}, {}, {"kernel": "direct", "phase": "fp64"}, {"coef": "f16"}, {"fafb": True},
                                {"top_k": 20, "full": False}]))
    if n_fd == 1:
        more["fd_lo"] = 0.0
    cap = 3.0e9 if more.get("kernel") == "direct" else 2.0e10
    while n_sft * n_sky * n_fd * n_f * more.get("units", 1) > cap:
        n_sky = max(1, n_sky // 2)
        if n_sky == 1:
            n_fd = max(1, n_fd // 2)
    return _unit(None, entry, n_sft, n_sky, n_fd, n_f, **more)


# ----------------------------------------------------------------- inputs
def _sizes(case):
    """Sizes of every work unit of the case; those of a batch are uneven, the
    first the largest."""
    keys = ("n_sft", "n_sky", "n_fd", "n_f", "dterms", "f0")
    first = {k: case[k] for k in keys}
    out = [first]
    for u in range(1, case["units"]):
        s = dict(first)
        if case["entry"] == "batch":
            r = np.random.Generator(np.random.PCG64(1000 * u + case["n_f"]))
            s["n_sft"] = max(4, int(case["n_sft"] * r.uniform(0.15, 1.0)))
            s["f0"] = round(float(r.uniform(50.0, 1500.0)), 3)
            if case["n_sky"] > 60:           # uneven grids; the wide units share one sky evenly
                s["n_sky"] = max(1, int(case["n_sky"] * r.uniform(0.125, 1.0)))
                s["n_f"] = max(64, int(case["n_f"] * r.uniform(0.125, 1.0)))
                s["n_fd"] = max(1, int(round(case["n_fd"] * r.uniform(0.25, 1.0))))
                s["dterms"] = int(r.choice([8, 16]))
        out.append(s)
    return out


def _t(x, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=dtype, device=DEV)


def _detectors(case, n_sft, gen, segment=0, of=1):
    """Start times (quantised to 2^-10 s, detector by detector) and the site of every SFT."""
    per = [n_sft // case["n_det"] + (d < n_sft % case["n_det"]) for d in range(case["n_det"])]
    t, site = [], []
    for d, n in enumerate(per):
        slots = max(n, int(math.ceil(n / case["keep"])))
        at = np.sort(gen.choice(slots, size=n, replace=False)) if slots > n else np.arange(n)
        x = EPOCH + (at + segment * slots) * T_SFT + (0.0 if slots > n else gen.uniform(0.0, 60.0, size=n))
        t.append(np.round(x * 1024.0) / 1024.0)
        site += [d] * n
    return np.concatenate(t), np.asarray(site, dtype=np.int32), np.concatenate([[0], np.cumsum(per)]).astype(np.int64)


EARTH = dict(t0=EPOCH, orbit_radius=ORBIT_R, orbit_rate=ORBIT_W, orbit_phase=0.3, obliquity=OBLIQUITY,
             earth_radius=EARTH_R, sidereal_rate=SIDEREAL_W, sidereal_phase=0.7)


def _geometry(t_mid, site):
    """Position, velocity (light-s, units of c) and arm tensor of every SFT, FP64 on the device."""
    dt = t_mid - EPOCH
    th = 0.3 + ORBIT_W * dt
    ce, se = math.cos(OBLIQUITY), math.sin(OBLIQUITY)
    lat, lon, ax, ay = (torch.tensor([s[k] for s in SITES], dtype=torch.float64, device=DEV)[site] for k in range(4))
    g = lon + 0.7 + SIDEREAL_W * dt
    c, s, cg, sg, cl, sl = torch.cos(th), torch.sin(th), torch.cos(g), torch.sin(g), torch.cos(lat), torch.sin(lat)
    z = torch.zeros_like(c)
    pos = ORBIT_R * torch.stack([c, s * ce, s * se], 1) + EARTH_R * torch.stack([cl * cg, cl * sg, sl], 1)
    vel = ORBIT_R * ORBIT_W * torch.stack([-s, c * ce, c * se], 1) + EARTH_R * SIDEREAL_W * cl[:, None] * torch.stack(
        [-sg, cg, z], 1)
    east, north = torch.stack([-sg, cg, z], 1), torch.stack([-sl * cg, -sl * sg, cl], 1)
    u, w = (torch.cos(a)[:, None] * north + torch.sin(a)[:, None] * east for a in (ax, ay))
    return pos, vel, 0.5 * (u[:, :, None] * u[:, None, :] - w[:, :, None] * w[:, None, :])


def _antenna(sky, tensor):
    """a, b [n_sky][n_sft] in FP64: the plus and cross projections on the wave frame."""
    rho = torch.sqrt(sky[:, 0] ** 2 + sky[:, 1] ** 2)
    ca, sa, zero = sky[:, 0] / rho, sky[:, 1] / rho, torch.zeros_like(rho)
    x = torch.stack([sa, -ca, zero], 1)
    y = torch.stack([-sky[:, 2] * ca, -sky[:, 2] * sa, rho], 1)
    flat = tensor.reshape(-1, 9).T.contiguous()

    def form(p, q):
        return (p[:, :, None] * q[:, None, :]).reshape(-1, 9) @ flat

    return form(x, x) - form(y, y), 2.0 * form(x, y)


def _sky(n):
    i = np.arange(n) + 0.5
    z = 1.0 - 2.0 * i / n if n > 1 else np.array([0.37])
    r, phi = np.sqrt(1.0 - z * z), math.pi * (3.0 - math.sqrt(5.0)) * i
    return np.stack([r * np.cos(phi), r * np.sin(phi), z], 1)


def _work_unit(case, s, gen, tgen, segment=0, sky_points=None, signals=()):
    """A work unit on the device; `signals`: (sky, spindown, frequency index, SNR, two complex amplitudes)."""
    t_start, site, offsets = _detectors(case, s["n_sft"], gen, segment)
    t_ref = EPOCH
    t0 = _t(t_start)
    site_d = torch.as_tensor(site, dtype=torch.int64, device=DEV)
    pos, vel, tensor = _geometry(t0 + 0.5 * T_SFT, site_d)
    sky = _t(_sky(s["n_sky"]) if sky_points is None else sky_points)
    a, b = (x.to(torch.float32).contiguous() for x in _antenna(sky, tensor))
    df = case["step"] / T_SFT
    fd0 = case["fd_lo"]
    dfd = -fd0 / (s["n_fd"] - 1) if s["n_fd"] > 1 else 0.0
    # the band that every template's frequency can reach, with the window
    v = 1.02 * (ORBIT_R * ORBIT_W + EARTH_R * SIDEREAL_W)
    tau = (-1.01 * ORBIT_R, float(t_start.max()) + T_SFT - t_ref + 1.01 * ORBIT_R)
    reach = [(f + fd * ta) * (1.0 + vv) * T_SFT for f in (s["f0"], s["f0"] + (s["n_f"] - 1) * df)
             for fd in (fd0, 0.0) for ta in tau for vv in (-v, v)]
    k_first = int(math.floor(min(reach))) - s["dterms"] - 2
    n_bins = int(math.floor(max(reach))) + s["dterms"] + 2 - k_first + 1
    x = torch.randn((s["n_sft"], n_bins, 2), generator=tgen, device=DEV) * math.sqrt(0.5)
    k = k_first + torch.arange(n_bins, dtype=torch.float64, device=DEV)
    for i_sky, i_fd, i_f, snr, p, q in signals:
        n = sky[i_sky]
        tt = (t0 + 0.5 * T_SFT - t_ref) + pos @ n
        f, fd = s["f0"] + i_f * df, fd0 + i_fd * dfd
        h = a[i_sky].double() * p + b[i_sky].double() * q
        h = h * (snr / torch.sqrt(2.0 * (h.abs() ** 2).sum()))
        phi = torch.remainder(tt * (f + 0.5 * fd * tt), 1.0)
        h = h * torch.exp(2j * math.pi * phi)
        at = (f + fd * tt) * (1.0 + vel @ n) * T_SFT
        wave = torch.sinc(at[:, None] - k[None, :]) * (1.0 - 2.0 * torch.remainder(k, 2.0))[None, :]
        x += torch.view_as_real(h[:, None] * wave).to(torch.float32)
    scale = None
    if case["storage"] != "c64":
        m = x.abs().amax(dim=(1, 2))
        scale = torch.where(m > 0, m / 256.0, torch.ones_like(m)).contiguous()
        x = (x / scale[:, None, None]).to(torch.bfloat16 if case["storage"] == "bf16" else torch.float16)
        x = x.view(torch.int16)
    return P.WorkUnit(n_det=case["n_det"], sft=x.contiguous(), sft_scale=scale, k_first=k_first, t_sft=T_SFT,
                      t_start=t0, pos=pos.contiguous(), vel=vel.contiguous(), sky=sky.contiguous(), a=a, b=b,
                      f0=s["f0"], df=df, n_f=s["n_f"], fdot0=fd0, dfdot=dfd, n_fd=s["n_fd"], t_ref=t_ref,
                      dterms=s["dterms"], det_offset=offsets)


def _threshold(n):
    """2F that about 150 of n noise templates exceed (chi-square, four degrees of freedom)."""
    x = 8.0
    while (1.0 + 0.5 * x) * math.exp(-0.5 * x) * n > 150.0:
        x += 0.25
    return x


def _units(case, seed):
    gen, tgen = np.random.Generator(np.random.PCG64(seed)), torch.Generator(device=DEV)
    tgen.manual_seed(seed)
    sizes = _sizes(case)

    def signal(s, snr):
        amp = gen.normal(size=4)
        return (int(gen.integers(s["n_sky"])), int(gen.integers(s["n_fd"])), int(gen.integers(s["n_f"])), snr,
                complex(amp[0], amp[1]), complex(amp[2], amp[3]))

    if case["entry"] == "semicoherent":
        signals = [signal(sizes[0], float(gen.uniform(4.0, 7.0))) for _ in range(2)]
        return [_work_unit(case, s, gen, tgen, segment=k, signals=signals) for k, s in enumerate(sizes)]
    wus = []
    points = _sky(10000)
    for s in sizes:
        shared = None                                    # a slice of one grid for the wide units
        if case["entry"] == "batch" and case["n_sky"] <= 60:
            shared = points[int(gen.integers(10000 - s["n_sky"])):][:s["n_sky"]]
        signals = [signal(s, float(gen.uniform(8.0, 20.0))) for _ in range(2)]
        wus.append(_work_unit(case, s, gen, tgen, sky_points=shared, signals=signals))
    return wus


def prepare(case, seed):
    if case["entry"] == "detector":
        gen = np.random.Generator(np.random.PCG64(seed))
        t_start, site, _ = _detectors(case, case["n_sft"], gen)
        v = gen.normal(size=(case["n_sky"], 3))
        n, m = case["n_sky"], case["n_sft"]
        out = dict(pos=torch.empty((m, 3), dtype=torch.float64, device=DEV),
                   vel=torch.empty((m, 3), dtype=torch.float64, device=DEV),
                   a=torch.empty((n, m), device=DEV), b=torch.empty((n, m), device=DEV))
        return dict(case=case, plan=P.Plan(max_sft=m, max_bins=1024, max_sky=n, max_fd=1, max_f=1),
                    t_mid=_t(t_start + 0.5 * T_SFT), site=torch.as_tensor(site, device=DEV),
                    sky=_t(v / np.linalg.norm(v, axis=1, keepdims=True)), out=out)
    wus = _units(case, seed)
    plan = P.Plan(max_sft=max(w.n_sft for w in wus), max_bins=max(w.n_bins for w in wus),
                  max_sky=max(w.n_sky for w in wus), max_fd=max(w.n_fd for w in wus), max_f=max(w.n_f for w in wus),
                  max_dterms=16, storage=case["storage"], phase=case["phase"], kernel=case["kernel"],
                  coef=case["coef"])
    outs = []
    for w in wus if case["entry"] != "semicoherent" else wus[:1]:
        shape = (w.n_sky, w.n_fd, w.n_f)
        o = P.Output(twoF=torch.empty(shape, device=DEV) if case["full"] else None)
        if case["fafb"]:
            o.fa, o.fb = torch.empty(shape + (2,), device=DEV), torch.empty(shape + (2,), device=DEV)
        if case["top_k"]:
            o.top_k, o.threshold = case["top_k"], _threshold(w.n_sky * w.n_fd * w.n_f)
            o.top = torch.empty((case["top_k"], 4), dtype=torch.int32, device=DEV)
            o.n_above = torch.empty(1, dtype=torch.int64, device=DEV)
        outs.append(o)
    return dict(case=case, plan=plan, wus=wus, outs=outs)


def _returned(o):
    r = dict(twoF=o.twoF, fa=o.fa, fb=o.fb)
    if o.top is not None:
        r.update(top_2F=o.top[:, :1].view(torch.float32), top_template=o.top[:, 1:], n_above=o.n_above)
    return r


def run(state):
    case, plan = state["case"], state["plan"]
    if case["entry"] == "detector":
        o = state["out"]
        plan.detector_inputs(EARTH, SITES, state["t_mid"], state["site"], state["sky"], o["pos"], o["vel"], o["a"],
                             o["b"])
        return o
    wus, outs = state["wus"], state["outs"]
    if case["entry"] == "compute":
        plan.compute(wus[0], outs[0])
    elif case["entry"] == "noalloc":
        plan.compute_noalloc(wus[0], outs[0])
    elif case["entry"] == "batch":
        plan.batch_compute(wus, outs)
    else:
        plan.semicoherent(wus, outs[0])
    return [_returned(o) for o in outs]


def work(case):
    """Each input read once and each output written once; per (template, SFT)
    pair a degree-7 complex polynomial, its phase factor, the rotation and two
    weighted sums (30 fused multiply-adds), or, for the term-by-term kernel,
    its loop over the window's terms."""
    if case["entry"] == "detector":
        m, n = case["n_sft"], case["n_sky"]
        return {"bytes": 12 * m + 24 * n + 48 * m + 8 * m * n, "flops": 40 * m * n}
    nbytes, flops = 0, 0
    for k, s in enumerate(_sizes(case)):
        n_bins = s["n_f"] * case["step"] + 2 * s["dterms"]
        templates = s["n_sky"] * s["n_fd"] * s["n_f"]
        nbytes += s["n_sft"] * n_bins * (8 if case["storage"] == "c64" else 4) + 56 * s["n_sft"]
        nbytes += 8 * s["n_sky"] * s["n_sft"] + 24 * s["n_sky"]
        if case["entry"] != "semicoherent" or k == 0:
            nbytes += templates * ((4 if case["full"] else 0) + (16 if case["fafb"] else 0)) + 16 * case["top_k"]
        per_pair = 2 * (10 * s["dterms"] + 28) if case["kernel"] == "direct" else 60
        flops += templates * s["n_sft"] * per_pair
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ exact
def _values(w, storage):
    x = w.sft.double() if storage == "c64" else w.sft.view(
        torch.bfloat16 if storage == "bf16" else torch.float16).double() * w.sft_scale.double()[:, None, None]
    return torch.view_as_complex(x.reshape(w.n_sft, w.n_bins, 2).contiguous())


def _exact_unit(w, storage):
    """2F, Fa, Fb of every template in FP64, term by term."""
    x = _values(w, storage)
    sign = 1.0 - 2.0 * torch.remainder(w.k_first + torch.arange(w.n_bins, dtype=torch.float64, device=DEV), 2.0)
    x = x * sign[None, :]                                # (-1)^k x[k]
    f = w.f0 + torch.arange(w.n_f, dtype=torch.float64, device=DEV) * w.df
    shape = (w.n_sky, w.n_fd, w.n_f)
    fa, fb = (torch.zeros(shape, dtype=torch.complex128, device=DEV) for _ in range(2))
    two_f = torch.zeros(shape, dtype=torch.float64, device=DEV)
    rows = max(1, 6_000_000 // w.n_f)
    for s in range(w.n_sky):
        n = w.sky[s]
        tau = (w.t_start + 0.5 * T_SFT - w.t_ref) + ((w.pos[:, 0] * n[0] + w.pos[:, 1] * n[1]) + w.pos[:, 2] * n[2])
        p = (1.0 + ((w.vel[:, 0] * n[0] + w.vel[:, 1] * n[1]) + w.vel[:, 2] * n[2])) * T_SFT
        a, b = w.a[s].double(), w.b[s].double()
        for i in range(w.n_fd):
            fd = w.fdot0 + i * w.dfdot
            for lo in range(0, w.n_sft, rows):
                r = slice(lo, min(w.n_sft, lo + rows))
                ta, pp = tau[r, None], p[r, None]
                at = f[None, :] * pp + (fd * ta) * pp
                k = torch.floor(at)
                kap = at - k
                col = (k - w.k_first).long()
                near = torch.sin(math.pi * torch.minimum(kap, 1.0 - kap)) / math.pi
                z = torch.zeros(at.shape, dtype=torch.complex128, device=DEV)
                for m in range(-w.dterms, w.dterms):
                    d = kap + m
                    weight = torch.where(d == 0, 1.0, near / d) * (1.0 if m % 2 == 0 else -1.0)
                    z += x[r].gather(1, col - m) * weight
                phi = torch.remainder(ta * (f[None, :] + (0.5 * fd) * ta), 1.0)
                z = z * torch.polar(torch.ones_like(phi), -2.0 * math.pi * phi)
                fa[s, i] += (a[r, None] * z).sum(0)
                fb[s, i] += (b[r, None] * z).sum(0)
        A, B, C = (a * a).sum(), (b * b).sum(), (a * b).sum()
        re = (fa[s] * fb[s].conj()).real
        two_f[s] = 2.0 * (B * fa[s].abs() ** 2 + A * fb[s].abs() ** 2 - 2.0 * C * re) / (A * B - C * C)
    return two_f, fa, fb


def exact(case, seed):
    if case["entry"] == "detector":
        st = prepare(case, seed)
        pos, vel, tensor = _geometry(st["t_mid"], st["site"].long())
        a, b = _antenna(st["sky"], tensor)
        return dict(pos=pos, vel=vel, a=a, b=b)
    sizes = _sizes(case)
    if sum(s["n_sky"] * s["n_fd"] * s["n_f"] * s["n_sft"] * s["dterms"] for s in sizes) > 5.0e10:
        return None                                      # minutes in FP64
    if sum(s["n_sky"] * s["n_fd"] for s in sizes) > 3000:
        return None
    got = [_exact_unit(w, case["storage"]) for w in _units(case, seed)]
    if case["entry"] == "semicoherent":
        got = [(sum(g[0] for g in got), None, None)]
    out = []
    for two_f, fa, fb in got:
        r = dict(twoF=two_f if case["full"] else None, fa=None, fb=None)
        if case["fafb"]:
            r.update(fa=torch.view_as_real(fa).contiguous(), fb=torch.view_as_real(fb).contiguous())
        if case["top_k"]:
            r.update(top_2F=torch.topk(two_f.reshape(-1), case["top_k"]).values[:, None], top_template=None,
                     n_above=None)
        out.append(r)
    return out
