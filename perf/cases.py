"""Timed cases of the aperture-mass path: what its users run, over the sizes
and options they run it at.

Each case is one pass through the package's public entry points on maps that
are already on the GPU.  Sizes are those of the repository's own workloads
(``synth``, ``bench.py``, ``tests``): maps of 16..4096 pixels a side, J planes,
R shear-randomised noise realisations, uneven batches of maps, fields of any
size with edges and missing pixels, and the direct sum the fast path is
compared with.

``listed`` holds the cases, ``draw`` more of the same ranges, ``prepare`` makes
a case's inputs from a seed, ``run`` is one pass, ``work`` the bytes and flops
a pass cannot do without, and ``exact`` the same results from plain torch in
float64.
"""
import math

import numpy as np
import torch

import paper_1204_4293_amd as amap

DEV = torch.device("cuda", 0)
DTYPES = {"f32": torch.float32, "f64": torch.float64}
SHAPE_NOISE = 0.3 / math.sqrt(20.0)  # per shear component
BOUNDARY = {"periodic": amap.BC_PERIODIC, "mirror": amap.BC_MIRROR, "zero": amap.BC_ZERO}
FILTER = {"starlet": amap.FILTER_STARLET, "s98": amap.FILTER_S98, "jbj04": amap.FILTER_JBJ04}
SIDES = (128, 256, 512, 1024, 2048)  # of an uneven batch, with the weights
SIDE_WEIGHTS = (4, 4, 3, 2, 1)       # of the repository's batch workload

_ctx = None


def context():
    """The one library context of the process, as a program keeps it."""
    global _ctx
    if _ctx is None:
        _ctx = amap.Context(0)
    return _ctx


def listed():
    return [
        # a cut-out looked at interactively in double precision: the smallest
        # call, all latency (KS and starlet of one 256^2 map)
        {"name": "map_256_f64", "kind": "map", "n": 256, "J": 5, "dtype": "f64", "rebuild": False},
        # the ordinary call: the aperture-mass maps of one 1024^2 shear map
        {"name": "map_1024_f32", "kind": "map", "n": 1024, "J": 7, "dtype": "f32", "rebuild": False},
        # a large map in double precision, decomposed and put together again
        # (the check a pipeline makes on its planes)
        {"name": "map_2048_f64", "kind": "map", "n": 2048, "J": 9, "dtype": "f64", "rebuild": True},
        # noise of one map from few realisations, as a served request of the
        # smallest size asks for it
        {"name": "noise_256_f32", "kind": "noise", "n": 256, "J": 6, "dtype": "f32", "R": 32},
        # the headline workload: sigma and S/N of a 1024^2 map from 256
        # realisations
        {"name": "noise_1024_f32", "kind": "noise", "n": 1024, "J": 7, "dtype": "f32", "R": 256},
        # the largest served request: 4096^2, 32 realisations
        {"name": "noise_4096_f32", "kind": "noise", "n": 4096, "J": 9, "dtype": "f32", "R": 32},
        # the whole path (signal, noise, S/N, peaks) in double precision, as a
        # validation run does it
        {"name": "path_1024_f64", "kind": "path", "n": 1024, "J": 8, "dtype": "f64", "R": 16},
        # a survey's tiles of uneven sizes through one kept batch plan
        {"name": "batch_48_f32", "kind": "batch", "maps": 48, "sides_seed": 31, "dtype": "f32"},
        # a survey field with edges, stars cut out: shear masked, inverted in a
        # zero-extended grid, decomposed under the mirror rule, peaks counted
        {"name": "field_1000_f32", "kind": "field", "ny": 1000, "nx": 1000, "P": 2048, "J": 7, "boundary": "mirror",
         "dtype": "f32"},
        # the noise of such a field
        {"name": "field_noise_1000_f32", "kind": "field_noise", "ny": 1000, "nx": 1000, "P": 2048, "J": 7,
         "boundary": "mirror", "dtype": "f32", "R": 16},
        # the brute-force aperture mass the fast path is compared with
        {"name": "direct_1024_f32", "kind": "direct", "n": 1024, "theta": 16.0, "filter": "starlet", "dtype": "f32"},
        # statistics of a map's S/N planes: peak counts, peak and trough
        # heights, moments
        {"name": "stats_1024_f32", "kind": "stats", "n": 1024, "planes": 6, "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("map", "map", "noise", "noise", "path", "batch", "field", "field_noise", "direct", "stats"))
    dtype = rng.choice(("f32", "f32", "f64"))
    if kind == "map":
        logn = rng.randint(4, 12 if dtype == "f32" else 11)
        return {"kind": kind, "n": 1 << logn, "J": rng.randint(2, min(logn, 10)), "dtype": dtype,
                "rebuild": rng.random() < 0.5}
    if kind == "noise":
        logn = rng.randint(5, 12)
        most = max(2, min(256, (1 << 28) >> (2 * logn)))
        return {"kind": kind, "n": 1 << logn, "J": rng.randint(min(logn, 4), min(logn, 9)), "dtype": "f32",
                "R": _log_int(rng, 2, most)}
    if kind == "path":
        logn = rng.randint(5, 10)
        return {"kind": kind, "n": 1 << logn, "J": rng.randint(min(logn, 4), min(logn, 8)), "dtype": "f64",
                "R": _log_int(rng, 2, 32 if logn < 10 else 16)}
    if kind == "batch":
        return {"kind": kind, "maps": _log_int(rng, 4, 60), "sides_seed": rng.randint(0, 1 << 20), "dtype": "f32"}
    if kind in ("field", "field_noise"):
        ny, nx = _log_int(rng, 40, 1024), _log_int(rng, 40, 1024)
        P = 16
        while P < max(ny, nx):
            P *= 2
        case = {"kind": kind, "ny": ny, "nx": nx, "P": P * rng.choice((1, 2)), "J": rng.randint(3, 8),
                "boundary": rng.choice(("mirror", "mirror", "zero", "periodic")), "dtype": dtype}
        if kind == "field_noise":
            case["R"] = _log_int(rng, 2, 16)
            case["dtype"] = "f32"
        return case
    if kind == "direct":
        n = 1 << rng.randint(8, 10)
        return {"kind": kind, "n": n, "theta": round(math.exp(rng.uniform(0.0, math.log(24.0))), 2),
                "filter": rng.choice(("starlet", "starlet", "s98", "jbj04")), "dtype": "f32"}
    return {"kind": kind, "n": 1 << rng.randint(5, 11), "planes": rng.randint(1, 8), "dtype": dtype}


# ---- inputs ------------------------------------------------------------------

def _generator(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFFFFFF)
    return g


def _frequencies(n):
    m = torch.arange(n, device=DEV)
    return torch.where(m < n // 2, m, m - n)


def _conj_d(n):
    """(real, imaginary) of conj(D(k)), D = [(k1^2 - k2^2) + 2 i nu k1 k2] / k^2."""
    m = _frequencies(n).to(torch.float64)
    m1, m2 = m[None, :], m[:, None]
    den = m1 * m1 + m2 * m2
    den[0, 0] = 1.0
    cross = 2.0 * m1 * m2
    cross[n // 2, :] = 0.0
    cross[:, n // 2] = 0.0
    return torch.complex((m1 * m1 - m2 * m2) / den, -cross / den)


def _shear(n, seed):
    """Shear of a Gaussian convergence field (P ~ k^-2, rms 0.02) with shape
    noise, float64."""
    g = _generator(seed)
    m = _frequencies(n).to(torch.float64)
    kk = torch.sqrt(m[None, :] ** 2 + m[:, None] ** 2)
    amp = torch.where(kk > 0, 1.0 / torch.clamp(kk, min=1.0), torch.zeros_like(kk))
    amp[n // 2, :] = 0.0
    amp[:, n // 2] = 0.0
    spec = torch.fft.fft2(torch.randn((n, n), generator=g, device=DEV, dtype=torch.float64)) * amp
    kappa = torch.fft.ifft2(spec).real
    spec = spec * (0.02 / torch.sqrt(torch.mean(kappa * kappa)))
    gamma = torch.fft.ifft2(spec * _conj_d(n).conj())
    noise = SHAPE_NOISE * torch.randn((2, n, n), generator=g, device=DEV, dtype=torch.float64)
    return gamma.real + noise[0], gamma.imag + noise[1]


def _maps(case, seed):
    """(g1, g2) of the case's map, or of its field (a corner of a map)."""
    dt = DTYPES[case["dtype"]]
    if "n" in case:
        g1, g2 = _shear(case["n"], seed)
    else:
        n = 16
        while n < max(case["ny"], case["nx"]):
            n *= 2
        g1, g2 = (g[:case["ny"], :case["nx"]] for g in _shear(n, seed))
    return g1.to(dt).contiguous(), g2.to(dt).contiguous()


def _mask(ny, nx, seed):
    """Observed pixels (1) of a field with stars cut out (about a tenth of it),
    one bad row and one bad column."""
    rng = np.random.default_rng(seed)
    m = np.ones((ny, nx), dtype=np.uint8)
    missing, target = 0, ny * nx // 10
    while missing < target:
        r = math.exp(rng.uniform(math.log(1.5), math.log(12.0)))
        cy, cx = rng.uniform(0, ny), rng.uniform(0, nx)
        y0, y1 = max(0, int(cy - r)), min(ny, int(cy + r) + 2)
        x0, x1 = max(0, int(cx - r)), min(nx, int(cx + r) + 2)
        yy, xx = np.mgrid[y0:y1, x0:x1]
        hit = ((yy - cy) ** 2 + (xx - cx) ** 2 <= r * r) & (m[y0:y1, x0:x1] != 0)
        m[y0:y1, x0:x1][hit] = 0
        missing += int(np.count_nonzero(hit))
    m[:, int(rng.integers(0, nx))] = 0
    m[int(rng.integers(0, ny)), :] = 0
    return torch.from_numpy(m).to(DEV)


def _sn_planes(count, ny, nx, dtype, seed):
    """S/N-like planes: unit-variance Gaussian fields smooth over 2^j pixels."""
    n = 16
    while n < max(ny, nx):
        n *= 2
    g = _generator(seed, 7)
    m = _frequencies(n).to(torch.float64) / n
    k2 = m[None, :] ** 2 + m[:, None] ** 2
    out = torch.empty((count, ny, nx), dtype=dtype, device=DEV)
    for j in range(count):
        # a band around the plane's scale, as a detail plane has
        s = 2.0 ** j
        band = torch.exp(-2.0 * (math.pi * s) ** 2 * k2 * 0.25) - torch.exp(-2.0 * (math.pi * s) ** 2 * k2)
        f = torch.fft.ifft2(torch.fft.fft2(torch.randn((n, n), generator=g, device=DEV, dtype=torch.float64)) * band).real
        out[j] = (f / torch.sqrt(torch.mean(f * f)))[:ny, :nx].to(dtype)
    return out


def _batch_sides(case):
    rng = np.random.default_rng(case["sides_seed"])
    w = np.array(SIDE_WEIGHTS, dtype=np.float64)
    return [int(s) for s in rng.choice(SIDES, size=case["maps"], p=w / w.sum())]


def prepare(case, seed):
    kind = case["kind"]
    ctx = context()
    st = {"case": case, "ctx": ctx, "noise_seed": int(seed) % 1000003 + 17}
    if kind == "batch":
        jobs = []
        for i, n in enumerate(_batch_sides(case)):
            g1, g2 = (g.to(DTYPES[case["dtype"]]) for g in _shear(n, seed * 64 + i))
            jobs.append({"g1": g1, "g2": g2,
                         "planes": torch.empty((n.bit_length() - 3, n, n), dtype=g1.dtype, device=DEV)})
        st["jobs"] = jobs
        st["plan"] = amap.BatchPlan(ctx, jobs)
        st["stream"] = torch.cuda.Stream()  # the plan replays a graph on it
        return st
    if kind == "stats":
        st["planes"] = _sn_planes(case["planes"], case["n"], case["n"], DTYPES[case["dtype"]], seed)
        return st
    st["g1"], st["g2"] = _maps(case, seed)
    if kind in ("noise", "field_noise"):
        # the planes of the signal, which S/N divides by sigma
        if kind == "noise":
            kappa, _ = ctx.ks_invert(st["g1"], st["g2"])
            st["signal"] = ctx.starlet_forward(kappa, case["J"])
        else:
            kappa, _ = ctx.ks_invert_padded(st["g1"], st["g2"], case["P"])
            st["signal"] = ctx.starlet_forward_bc(kappa, case["J"], BOUNDARY[case["boundary"]])
    if kind == "field":
        st["mask"] = _mask(case["ny"], case["nx"], seed)
        st["snr"] = _sn_planes(case["J"] - 1, case["ny"], case["nx"], st["g1"].dtype, seed)
    return st


# ---- one pass ----------------------------------------------------------------

def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["case"]["kind"]
    if kind == "map":
        kappa, _ = ctx.ks_invert(st["g1"], st["g2"])
        planes = ctx.starlet_forward(kappa, case["J"])
        out = {"kappa_e": kappa, "planes": planes}
        if case["rebuild"]:
            out["rebuilt"] = ctx.starlet_reconstruct(planes)
        return out
    if kind == "noise":
        sigma, snr = ctx.noise_maps(st["g1"], st["g2"], case["J"], case["R"], st["noise_seed"],
                                    planes_signal=st["signal"])
        return {"sigma": sigma, "snr": snr}
    if kind == "path":
        return ctx.run_path(st["g1"], st["g2"], case["J"], case["R"], st["noise_seed"], 3.0)
    if kind == "batch":
        with torch.cuda.stream(st["stream"]):
            st["plan"].run()
        return [j["planes"] for j in st["jobs"]]
    if kind == "field":
        bc = BOUNDARY[case["boundary"]]
        g1, g2 = ctx.mask_shear(st["g1"], st["g2"], st["mask"])
        kappa, _ = ctx.ks_invert_padded(g1, g2, case["P"])
        planes = ctx.starlet_forward_bc(kappa, case["J"], bc)
        peaks = ctx.count_peaks_masked(st["snr"], st["mask"], 3.0, bc)
        return {"g1": g1, "g2": g2, "kappa_e": kappa, "planes": planes, "peaks": peaks}
    if kind == "field_noise":
        sigma, snr = ctx.noise_maps_bc(st["g1"], st["g2"], case["P"], case["J"], BOUNDARY[case["boundary"]],
                                       case["R"], st["noise_seed"], planes_signal=st["signal"])
        return {"sigma": sigma, "snr": snr}
    if kind == "direct":
        return ctx.map_direct(st["g1"], st["g2"], case["theta"], FILTER[case["filter"]], fparam=_fparam(case))
    planes = st["planes"]
    return {"peaks": ctx.count_peaks(planes, 3.0),
            "heights": ctx.peak_histogram(planes, -2.0, 6.0, 40),
            "depths": ctx.peak_histogram(planes, -2.0, 6.0, 40, sign=-1),
            "moments": ctx.plane_moments(planes)}


def _fparam(case):
    return {"starlet": 0.0, "s98": 1.0, "jbj04": 0.5}[case["filter"]]


# ---- what a pass cannot do without ---------------------------------------------

def work(case):
    """Inputs read once and outputs written once; flops of the method (5 m log2
    m a complex transform of m points, 19 a pixel and starlet scale, 50 a
    pixel for a random rotation, 4 a pixel and scale for running statistics)."""
    e = 4.0 if case["dtype"] == "f32" else 8.0
    kind = case["kind"]

    def ks(n):
        return 20.0 * n * n * math.log2(n) + 6.0 * n * n

    if kind == "batch":
        b = f = 0.0
        for n in _batch_sides(case):
            J = n.bit_length() - 3
            b += e * n * n * (2 + J)
            f += ks(n) + 19.0 * n * n * (J - 1)
        return {"bytes": b, "flops": f}
    if kind in ("field", "field_noise"):
        p, J, P = float(case["ny"] * case["nx"]), case["J"], case["P"]
        if kind == "field":
            # shear and mask, S/N planes in; masked shear, kappa, planes out
            return {"bytes": p * (e * (2 + (J - 1) + 3 + J) + 1.0), "flops": ks(P) + 19.0 * p * (J - 1)}
        one = ks(P) + 50.0 * p + 23.0 * p * (J - 1)
        return {"bytes": e * p * (2 + (J - 1) + 2 * (J - 1)), "flops": case["R"] * one}
    n = case["n"]
    p = float(n * n)
    if kind == "map":
        J, again = case["J"], bool(case["rebuild"])
        return {"bytes": e * p * (2 + 1 + J + again), "flops": ks(n) + (19.0 + again) * p * (J - 1)}
    if kind in ("noise", "path"):
        J = case["J"]
        one = ks(n) + 50.0 * p + 23.0 * p * (J - 1)
        if kind == "noise":
            return {"bytes": e * p * (2 + (J - 1) + 2 * (J - 1)), "flops": case["R"] * one}
        return {"bytes": e * p * (2 + 1 + J + 2 * (J - 1)), "flops": case["R"] * one + ks(n) + 19.0 * p * (J - 1)}
    if kind == "direct":
        return {"bytes": e * p * 3, "flops": 4.0 * p * math.pi * _cut(case) ** 2}
    return {"bytes": e * p * case["planes"], "flops": 40.0 * p * case["planes"]}


def _cut(case):
    return case["theta"] * {"starlet": 2.0, "s98": 1.0, "jbj04": 5.0}[case["filter"]]


# ---- the same results from plain torch in float64 --------------------------------

def _ks(g1, g2, conj_d):
    return torch.fft.ifft2(torch.fft.fft2(torch.complex(g1, g2)) * conj_d).real


def _taps(n, d, boundary):
    """Index of the five taps of every sample (-1: a sample that is 0)."""
    i = torch.arange(n, device=DEV)[None, :] + d * torch.arange(-2, 3, device=DEV)[:, None]
    if boundary == "periodic":
        return i % n
    if boundary == "mirror":
        k = i % (2 * (n - 1))
        return torch.where(k < n, k, 2 * (n - 1) - k)
    return torch.where((i >= 0) & (i < n), i, torch.full_like(i, -1))


def _smooth(c, d, boundary):
    ty, tx = _taps(c.shape[0], d, boundary), _taps(c.shape[1], d, boundary)
    h = (0.0625, 0.25, 0.375, 0.25, 0.0625)
    row = sum(w * c[:, t.clamp(min=0)] * (t >= 0) for w, t in zip(h, tx))
    return sum(w * row[t.clamp(min=0), :] * (t >= 0)[:, None] for w, t in zip(h, ty))


def _starlet(c, J, boundary="periodic"):
    out = []
    for j in range(1, J):
        nxt = _smooth(c, 1 << (j - 1), boundary)
        out.append(c - nxt)
        c = nxt
    out.append(c)
    return torch.stack(out)


def _angles(count, seed, r):
    """2 pi u of the `count` pixels of realisation r: Philox4x64-10, key
    (seed, 0), block counters (b, r, 0, 0), each 64-bit word low half first."""
    bg = np.random.Philox(key=int(seed), counter=((int(r) << 64) - 1) % (1 << 256))
    words = bg.random_raw(4 * ((count + 7) // 8)).view(np.uint32)[:count]
    v = torch.from_numpy((words >> np.uint32(8)).astype(np.int32)).to(DEV)
    return v.to(torch.float64) * (2.0 * math.pi * 2.0 ** -24)


def _noise(g1, g2, J, R, seed, conj_d, P, boundary):
    """sigma over R realisations of the field in a P x P grid (Welford)."""
    ny, nx = g1.shape
    mean = m2 = 0.0
    grid = torch.zeros((P, P), dtype=torch.complex128, device=DEV)
    for r in range(R):
        turn = _angles(ny * nx, seed, r).reshape(ny, nx)
        grid[:ny, :nx] = torch.complex(g1, g2) * torch.polar(torch.ones_like(turn), turn)
        kappa = torch.fft.ifft2(torch.fft.fft2(grid) * conj_d).real[:ny, :nx]
        w = _starlet(kappa, J, boundary)[:-1]
        d = w - mean
        mean = mean + d / (r + 1)
        m2 = m2 + d * (w - mean)
    return torch.sqrt(m2 / (R - 1))


def _divide(w, sigma):
    return torch.where(sigma > 0, w / torch.where(sigma > 0, sigma, torch.ones_like(sigma)), torch.zeros_like(w))


def _q_starlet(x):
    e, e2 = x, x * x

    def c3(v):
        return abs(v) ** 3

    if e == 0.0:
        return 0.0
    return (-279.0 * e2 * c3(e) + 8.0 * (1 + 6 * e + 24 * e2) * c3(0.5 - e) - 9.0 * (1 + 3 * e + 6 * e2) * c3(1 - e)
            - 9.0 * (1 - 3 * e + 6 * e2) * c3(1 + e) + (1 + 1.5 * e + 1.5 * e2) * c3(2 - e)
            + (1 - 1.5 * e + 1.5 * e2) * c3(2 + e) + 8.0 * (1 - 6 * e + 24 * e2) * c3(0.5 + e)) / (45.0 * e2)


def _q(case, r):
    theta, x2 = case["theta"], (r / case["theta"]) ** 2
    if case["filter"] == "starlet":
        return _q_starlet(r / theta) / theta ** 2
    p = _fparam(case)
    if case["filter"] == "s98":
        return (1 + p) * (2 + p) / (math.pi * theta ** 2) * x2 * (1 - x2) ** p if r <= theta else 0.0
    return p * x2 * math.exp(-p * x2) / theta ** 2


def _direct(case, g1, g2):
    """The sum as a periodic convolution with the tabulated weights."""
    n, cut = case["n"], _cut(case)
    R = int(math.floor(cut))
    wc, ws = np.zeros((n, n)), np.zeros((n, n))
    for dy in range(-R, R + 1):
        for dx in range(-R, R + 1):
            r2 = float(dx * dx + dy * dy)
            if r2 == 0.0 or r2 > cut * cut:
                continue
            q = _q(case, math.sqrt(r2))
            wc[-dy % n, -dx % n] = q * (dx * dx - dy * dy) / r2
            ws[-dy % n, -dx % n] = q * 2.0 * dx * dy / r2
    f = torch.fft.rfft2
    wc, ws = torch.from_numpy(wc).to(DEV), torch.from_numpy(ws).to(DEV)
    return -torch.fft.irfft2(f(g1) * f(wc) + f(g2) * f(ws), s=(n, n))


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for i, n in enumerate(_batch_sides(case)):
            g1, g2 = (g.to(DTYPES[case["dtype"]]).double() for g in _shear(n, seed * 64 + i))
            out.append(_starlet(_ks(g1, g2, _conj_d(n)), n.bit_length() - 3))
        return out
    if kind == "stats":
        x = _sn_planes(case["planes"], case["n"], case["n"], DTYPES[case["dtype"]], seed).double()
        mean = x.mean(dim=(1, 2))
        d = x - mean[:, None, None]
        m = torch.stack([mean] + [(d ** k).mean(dim=(1, 2)) for k in (2, 3, 4)], dim=1)
        return {"peaks": None, "heights": None, "depths": None, "moments": m}
    g1, g2 = _maps(case, seed)
    noise_seed = int(seed) % 1000003 + 17
    if kind == "field":
        mask = _mask(case["ny"], case["nx"], seed) != 0
        g1, g2 = (torch.where(mask, g, torch.zeros_like(g)) for g in (g1, g2))
    masked = (g1, g2)
    g1, g2 = g1.double(), g2.double()
    if kind == "direct":
        return _direct(case, g1, g2)
    if kind in ("field", "field_noise"):
        P, J, bc = case["P"], case["J"], case["boundary"]
        cd = _conj_d(P)
        grid = torch.zeros((2, P, P), dtype=torch.float64, device=DEV)
        grid[0, :case["ny"], :case["nx"]], grid[1, :case["ny"], :case["nx"]] = g1, g2
        kappa = _ks(grid[0], grid[1], cd)[:case["ny"], :case["nx"]]
        planes = _starlet(kappa, J, bc)
        if kind == "field":
            return {"g1": masked[0], "g2": masked[1], "kappa_e": kappa, "planes": planes, "peaks": None}
        sigma = _noise(g1, g2, J, case["R"], noise_seed, cd, P, bc)
        return {"sigma": sigma, "snr": _divide(planes[:-1], sigma)}
    cd = _conj_d(case["n"])
    kappa = _ks(g1, g2, cd)
    planes = _starlet(kappa, case["J"])
    if kind == "map":
        out = {"kappa_e": kappa, "planes": planes}
        if case["rebuild"]:
            out["rebuilt"] = kappa
        return out
    sigma = _noise(g1, g2, case["J"], case["R"], noise_seed, cd, case["n"], "periodic")
    out = {"sigma": sigma, "snr": _divide(planes[:-1], sigma)}
    if kind == "path":
        out.update(kappa_e=kappa, planes=planes, peaks=None)
    return out
