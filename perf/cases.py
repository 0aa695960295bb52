"""The calls whose time matters to a user of this library, over the sizes they are used at.

One case is one call (or one short sequence of calls) of the public binding: a transform, a pair of
transforms, a messenger solve of one map or of a batch, a polarised solve, a band-limited schedule,
an uneven group, a burst of served requests. Sizes follow the library's own workloads and tests:
Nside 16 / lmax 32 (the small band problem) up to Nside 1024 / lmax 2048 (the precision problem),
the satellite problem at Nside 512 / lmax 1024, batches of up to 64 simulations, odd band limits up
to 4 Nside - 1. Solves run a shortened cooling schedule: every sweep does the same work, so a few
show what a full schedule of 80 to 140 costs.

Data are a random field of plane waves with the amplitudes of the problem's spectrum plus white
noise of the pixels' variance, made on the GPU from the seed alone. `exact` evaluates the same calls
from the definitions in plain torch, in 64 bits.
"""
import functools
import math

import numpy as np
import torch

from paper_1211_0585_amd import mwf

DTYPES = {"f64": mwf.WF_F64, "f32": mwf.WF_F32, "bf16x6": mwf.WF_BF16X6, "bf16x3": mwf.WF_BF16X3}

# members of the uneven group and the served burst: maps@(Nside, lmax) and Nside of each request
GROUP = ((32, 128, 256), (16, 256, 512), (8, 512, 1024))
SERVED = (64, 128, 256, 64, 128, 256)


def listed():
    return [
        # one small forward transform: launches and latency, nothing else
        {"name": "analysis_small", "kind": "analysis", "dtype": "f64", "nside": 16, "lmax": 32, "maps": 1},
        # one inverse transform at an odd band limit of 3 Nside - 1
        {"name": "synthesis_odd", "kind": "synthesis", "dtype": "f64", "nside": 64, "lmax": 191, "maps": 1},
        # the small band problem: a solve that is all launches
        {"name": "solve_small", "kind": "solve", "dtype": "f64", "nside": 16, "lmax": 32, "maps": 1, "sweeps": 20},
        # the satellite problem, one map, plain FP64: the headline workload
        {"name": "solve_satellite", "kind": "solve", "dtype": "f64", "nside": 512, "lmax": 1024, "maps": 1,
         "sweeps": 8},
        # the largest transform pair: synthesis of a sky and its analysis
        {"name": "pair_large", "kind": "pair", "dtype": "f64", "nside": 1024, "lmax": 2048, "maps": 1},
        # 64 simulations sharing one noise model, FP32 matrix cores: the batched workload
        {"name": "batch_f32", "kind": "solve", "dtype": "f32", "nside": 512, "lmax": 1024, "maps": 64, "sweeps": 4},
        # a smaller batch through the split-bf16 matrix path, odd band limit
        {"name": "batch_bf16x6", "kind": "solve", "dtype": "bf16x6", "nside": 256, "lmax": 511, "maps": 16,
         "sweeps": 6},
        # the precision problem: one large map in FP32
        {"name": "solve_f32_large", "kind": "solve", "dtype": "f32", "nside": 1024, "lmax": 2048, "maps": 1,
         "sweeps": 3},
        # temperature and polarisation together
        {"name": "polarised", "kind": "pol", "dtype": "f64", "nside": 512, "lmax": 1024, "maps": 1, "sweeps": 3},
        # the cooling schedule with band-limited transforms (levels as the adaptive solve picks them)
        {"name": "banded", "kind": "banded", "dtype": "f64", "nside": 512, "lmax": 1024, "maps": 1, "sweeps": 10},
        # uneven batch: plans of three sizes stepped together
        {"name": "group_uneven", "kind": "group", "dtype": "f32", "nside": 512, "lmax": 1024, "maps": 56,
         "sweeps": 4},
        # a burst of requests to a running server, host arrays in and out
        {"name": "served_burst", "kind": "served", "dtype": "f32", "nside": 256, "lmax": 512, "maps": 6, "sweeps": 8},
    ]


def draw(rng):
    """One more case of the same ranges: Nside 8..1024, any band limit a plan takes, 1..64 maps."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(("analysis", "synthesis", "pair", "solve", "solve", "solve", "pol", "banded"))
        dtype = rng.choice(("f64", "f64", "f32", "bf16x6", "bf16x3"))
        nside = 2 ** rng.randint(3, 10)
        lmax = int(round(math.exp(rng.uniform(math.log(nside), math.log(4 * nside - 1)))))
        maps = int(round(math.exp(rng.uniform(0.0, math.log(64)))))
        if kind == "pol":
            dtype, nside, maps = "f64", min(nside, 512), 1 + maps % 2
        if kind == "banded":
            maps = 1
        elif dtype == "f64" and kind != "pol":
            maps = 1 + maps % 4
        case = {"kind": kind, "dtype": dtype, "nside": nside, "lmax": min(lmax, 4 * nside - 1, 2048), "maps": maps}
        if kind in ("solve", "pol", "banded"):
            case["sweeps"] = rng.randint(2, 8)
        if work(case)["flops"] <= 0.5 * most and maps * nside * nside <= 64 * 512 * 512:
            return case


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=None)
def rings(nside):
    """Iso-latitude rings in RING order: z, pixels, first pixel, and ph in phi_j = pi (ph + 2 j) / pixels."""
    i = np.arange(1, 4 * nside)
    cap = np.minimum(i, 4 * nside - i)
    polar = cap < nside
    zc = 1.0 - cap.astype(np.float64) ** 2 / (3.0 * nside * nside)
    z = np.where(polar, np.where(i < 2 * nside, zc, -zc), 2.0 * (2 * nside - i) / (3.0 * nside))
    n = np.where(polar, 4 * cap, 4 * nside)
    ph = np.where(polar, 1, (i - nside + 1) % 2)
    start = np.concatenate([[0], np.cumsum(n)[:-1]])
    return z, n, start, ph


def _directions(nside):
    """Unit vectors of the pixels, [npix, 3] on the GPU."""
    z, n, start, ph = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in rings(nside))
    r = torch.repeat_interleave(torch.arange(len(n), device="cuda"), n)
    j = torch.arange(len(r), device="cuda") - start[r]
    phi = math.pi * (ph[r] + 2 * j).double() / n[r]
    zr = z[r]
    st = torch.sqrt((1.0 - zr) * (1.0 + zr))
    return torch.stack([st * torch.cos(phi), st * torch.sin(phi), zr], 1)


def _spectrum(lmax):
    l = np.arange(lmax + 1, dtype=np.float64)
    cl = np.zeros(lmax + 1)
    bump = 1.0 + sum(0.6 * np.exp(-(l - k) ** 2 / 7200.0) for k in (220.0, 540.0, 800.0))
    s = math.radians(13.0 / 60.0) / math.sqrt(8.0 * math.log(2.0))
    cl[2:] = 1e3 / (l[2:] * (l[2:] + 1.0)) * bump[2:] * np.exp(-l[2:] * (l[2:] + 1.0) * s * s)
    return cl


def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000 + stream)


def _sky(nside, lmax, maps, seed, dtype):
    """[maps, npix]: sums of 24 plane waves with wave numbers up to lmax, rms about that of the spectrum."""
    g = _generator(seed, 1)
    v = _directions(nside)
    out = torch.empty((maps, v.shape[0]), dtype=dtype, device="cuda")
    top = math.log(max(4.0, lmax))
    for i in range(maps):
        k = torch.exp(math.log(2.0) + (top - math.log(2.0)) * torch.rand(24, generator=g, device="cuda", dtype=torch.float64))
        d = torch.randn(3, 24, generator=g, device="cuda", dtype=torch.float64)
        a = 18.0 * torch.randn(24, generator=g, device="cuda", dtype=torch.float64)
        p = 2.0 * math.pi * torch.rand(24, generator=g, device="cuda", dtype=torch.float64)
        f = torch.zeros(v.shape[0], dtype=torch.float64, device="cuda")
        w = k * d / d.norm(dim=0)
        for c in range(24):
            f += a[c] * torch.cos(v[:, 0] * w[0, c] + v[:, 1] * w[1, c] + v[:, 2] * w[2, c] + p[c])
        out[i] = f
    return out


def _noise(nside, seed, bcut_deg=15.0, scale=1.0):
    """(sigma^2, mask True where cut) per pixel: scan-weighted hits times a log-normal scatter, galactic cut."""
    g = _generator(seed, 2)
    v = _directions(nside)
    b, l = math.radians(29.81), math.radians(96.38)
    ce = v[:, 0] * (math.cos(b) * math.cos(l)) + v[:, 1] * (math.cos(b) * math.sin(l)) + v[:, 2] * math.sin(b)
    hits = 300.0 * (1.0 + 2.0 * ce.abs() ** 4) * torch.exp(
        0.2 * torch.randn(v.shape[0], generator=g, device="cuda", dtype=torch.float64))
    sigma2 = (2200.0 * scale * nside / 512.0) ** 2 / hits
    return sigma2, v[:, 2].abs() < math.sin(math.radians(bcut_deg))


def _schedule(sweeps):
    """Geometric cooling 1e4 -> 1 over the first half, then lambda = 1."""
    c = max(1, sweeps // 2)
    k = np.arange(c)
    return np.concatenate([1e4 ** (1.0 - k / c), np.ones(sweeps - c)])


def _bands(lmax, sweeps):
    """Band limits of a cooling schedule: four truncated levels over the first half, the full band after."""
    h = sweeps // 2
    levels = [min(lmax, b) for b in (120, 140, 180, 260)]
    return np.array([levels[min(3, 4 * k // max(1, h))] if k < h else lmax for k in range(sweeps)], dtype=np.int32)


def _real(dtype):
    return torch.float64 if dtype == "f64" else torch.float32


def _problem(nside, lmax, maps, seed, dtype, bcut_deg=15.0, scale=1.0):
    """(C_l, N^-1 with zeros where cut, data [maps, npix]) of a solve."""
    sigma2, cut = _noise(nside, seed, bcut_deg, scale)
    d = _sky(nside, lmax, maps, seed, torch.float64)
    g = _generator(seed, 3)
    sd = torch.sqrt(sigma2)
    for i in range(maps):
        d[i] += sd * torch.randn(sd.shape[0], generator=g, device="cuda", dtype=torch.float64)
    ninv = torch.where(cut, torch.zeros_like(sigma2), 1.0 / sigma2)
    return _spectrum(lmax), ninv, d.to(dtype)


def _alm(lmax, maps, seed, dtype, cl):
    """[maps, N_lm] random alm of the spectrum cl in packed order (m-major)."""
    g = _generator(seed, 4)
    m, l = _packed(lmax)
    x = torch.randn((maps, len(l), 2), generator=g, device="cuda", dtype=torch.float64)
    x *= torch.from_numpy(np.sqrt(0.5 * cl[l])).cuda()[None, :, None]
    x[:, :lmax + 1, 0] *= math.sqrt(2.0)
    x[:, :lmax + 1, 1] = 0.0
    return torch.view_as_complex(x).to(torch.complex128 if dtype == torch.float64 else torch.complex64).contiguous()


@functools.lru_cache(maxsize=None)
def _packed(lmax):
    m = np.repeat(np.arange(lmax + 1), np.arange(lmax + 1, 0, -1))
    l = np.concatenate([np.arange(k, lmax + 1) for k in range(lmax + 1)])
    return m, l


def _pol_problem(nside, lmax, maps, seed):
    """(spectra [4, lmax+1], N^-1 [6, npix], mask bytes, data [maps, 3, npix]) of a polarised solve."""
    sigma2, cut = _noise(nside, seed)
    g = _generator(seed, 5)
    rho = 0.6 * torch.rand(sigma2.shape[0], generator=g, device="cuda", dtype=torch.float64) - 0.3
    sp = 2.0 * sigma2
    det = sp * sp * (1.0 - rho * rho)
    z = torch.zeros_like(sp)
    ninv6 = torch.stack([1.0 / sigma2, sp / det, sp / det, z, z, -rho * sp / det])
    v = _directions(nside)
    cut_p = v[:, 2].abs() < math.sin(math.radians(20.0))
    bits = (~cut).to(torch.uint8) | ((~cut_p).to(torch.uint8) << 1)
    tt = _spectrum(lmax)
    l = np.arange(lmax + 1)
    ee = 0.05 * tt
    te = 0.5 * np.cos(np.pi * l / 150.0) * np.sqrt(tt * ee)
    cl4 = np.stack([tt, ee, 0.01 * ee, te])
    d = _sky(nside, lmax, 3 * maps, seed, torch.float64).view(maps, 3, -1)
    d[:, 1:] *= 0.2
    sd = torch.stack([sigma2, sp, sp]).sqrt()
    for i in range(maps):
        n = torch.randn(sd.shape, generator=g, device="cuda", dtype=torch.float64)
        n[2] = rho * n[1] + torch.sqrt(1.0 - rho * rho) * n[2]
        d[i] += sd * n
    return cl4, ninv6, bits, d


def _request(k, nside, seed):
    """Request k of the served burst: its own galactic cut and noise level."""
    cl, ninv, d = _problem(nside, 2 * nside, 1, 97 * seed + k, torch.float64, 5.0 + 4.0 * k, 0.3 + 0.2 * k)
    return cl, ninv, d[0]


# ------------------------------------------------------------------ the calls
def prepare(case, seed):
    kind, nside, lmax, maps = case["kind"], case["nside"], case["lmax"], case["maps"]
    rt, dt = _real(case["dtype"]), DTYPES[case["dtype"]]
    st = {"kind": kind, "lam": _schedule(case.get("sweeps", 1))}
    if kind == "pol":
        cl4, ninv6, bits, d = _pol_problem(nside, lmax, maps, seed)
        st["plan"] = mwf.PolPlan(nside, lmax, cl4, ninv6.cpu().numpy(), bits.cpu().numpy(), max_batch=maps)
        st["d"] = d if maps > 1 else d[0]
        return st
    if kind == "group":
        st["plans"], st["d"] = [], []
        for k, (n, ns, lm) in enumerate(GROUP):
            cl, ninv, d = _problem(ns, lm, n, 31 * seed + k, rt)
            st["plans"].append(mwf.Plan(ns, lm, cl, ninv.cpu().numpy(), dtype=dt, max_batch=n))
            st["d"].append(d)
        st["group"] = mwf.Group(st["plans"], [n for n, _, _ in GROUP])
        st["group"].autotune(st["d"])
        return st
    if kind == "served":
        st["server"] = mwf.Server(hbm_budget=8 << 30, max_slots=16)
        st["requests"] = []
        for k, ns in enumerate(SERVED):
            cl, ninv, d = _request(k, ns, seed)
            st["requests"].append((ns, 2 * ns, cl, ninv.cpu().numpy(), d.cpu().numpy()))
        # a running server has served these shapes before
        for t in [st["server"].submit(*st["requests"][k], np.ones(1)) for k in range(3)]:
            st["server"].wait(t)
        return st
    cl, ninv, d = _problem(nside, lmax, maps, seed, rt)
    st["plan"] = mwf.Plan(nside, lmax, cl, ninv.cpu().numpy(), dtype=dt, max_batch=maps)
    if dt != mwf.WF_F64:
        st["plan"].autotune(maps)
    st["d"] = d if maps > 1 else d[0]
    if kind in ("synthesis", "pair"):
        a = _alm(lmax, maps, seed, rt, cl)
        st["alm"] = a if maps > 1 else a[0]
    if kind == "banded":
        st["bands"] = _bands(lmax, case["sweeps"])
    return st


def run(st):
    kind = st["kind"]
    if kind == "analysis":
        return st["plan"].map2alm(st["d"])
    if kind == "synthesis":
        return st["plan"].alm2map(st["alm"])
    if kind == "pair":
        m = st["plan"].alm2map(st["alm"])
        return m, st["plan"].map2alm(m)
    if kind == "banded":
        return st["plan"].solve_banded(st["d"], st["lam"], st["bands"])
    if kind == "group":
        return st["group"].solve(st["d"], st["lam"])
    if kind == "served":
        s = st["server"]
        tickets = [s.submit(*r, st["lam"]) for r in st["requests"]]
        # served maps carry FP32 results: kept as such
        return [s.wait(t)[0].astype(np.float32) for t in tickets]
    return st["plan"].solve(st["d"], st["lam"])


# ------------------------------------------------------------------ work
def _members(case):
    if case["kind"] == "group":
        return [(n, ns, lm) for n, ns, lm in GROUP]
    if case["kind"] == "served":
        return [(1, ns, 2 * ns) for ns in SERVED]
    return [(case["maps"] * (3 if case["kind"] == "pol" else 1), case["nside"], case["lmax"])]


def work(case):
    """Per transform of one real map: a multiply-add of the real and the imaginary part per (l, m, ring pair), and
    a real FFT of every ring. A polarised map counts three spin-0 ones, its E and B sums twice (two functions each).
    A sweep is a pair of transforms and Eq. (3) per pixel; d, N^-1 and the results pass memory once."""
    kind = case["kind"]
    el = 8 if case["dtype"] == "f64" else 4
    flops = bytes_ = 0.0
    bands = _bands(case["lmax"], case["sweeps"]) if kind == "banded" else None
    for n, ns, lm in _members(case):
        npix, nalm = 12.0 * ns * ns, 0.5 * (lm + 1) * (lm + 2)
        sht = lambda L: 4.0 * 2 * ns * 0.5 * (L + 1) * (L + 2) * (5.0 / 3.0 if kind == "pol" else 1.0)  # noqa: E731
        fft = 2.5 * npix * math.log2(4 * ns)
        if kind in ("analysis", "synthesis", "pair"):
            t = 2 if kind == "pair" else 1
            flops += n * t * (sht(lm) + fft)
            bytes_ += n * t * (npix + 2 * nalm) * el
        else:
            for k in range(case["sweeps"]):
                flops += n * (2 * (sht(int(bands[k]) if bands is not None else lm) + fft) + 6 * npix)
            noise = 2 * npix if kind == "pol" else npix
            bytes_ += (n * (2 * npix + 2 * nalm) + noise) * el
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------------------ the same calls from the definitions, 64 bits
class _Sphere:
    """Transform pair of [columns] real maps at (nside, lmax): Fourier sums along the rings by their matrices,
    Legendre sums over ring pairs with every m stepped in l together."""

    STEPS = 16     # values of l per batched product

    def __init__(self, nside, lmax):
        self.nside, self.lmax = nside, lmax
        z, n, start, ph = rings(nside)
        self.q = 2 * nside                                  # north rings and the equator, ring 0 first
        self.n, self.start, self.ph = n, start, ph
        self.omega = 4.0 * math.pi / (12 * nside * nside)
        self.z_np = z[:self.q]
        self.z = torch.from_numpy(np.ascontiguousarray(self.z_np)).cuda()

    def _phases(self, n, ph):
        t = torch.arange(2 * n, device="cuda", dtype=torch.float64) * (math.pi / n)
        j = (ph + 2 * torch.arange(n, device="cuda")) % (2 * n)
        idx = (j[:, None] * torch.arange(self.lmax + 1, device="cuda")[None, :]) % (2 * n)
        return torch.cos(t)[idx], torch.sin(t)[idx]          # [n, lmax + 1]

    def _ring_sets(self):
        """Ring pairs that share a matrix: (n, ph, list of north rings)."""
        sets = {}
        for r in range(self.q):
            sets.setdefault((int(self.n[r]), int(self.ph[r])), []).append(r)
        return sets

    def _pixels(self, rs, n):
        south = [4 * self.nside - 2 - r for r in rs]
        j = torch.arange(n, device="cuda")
        a = torch.from_numpy(self.start[rs]).cuda()[:, None] + j
        b = torch.from_numpy(self.start[south]).cuda()[:, None] + j
        return a, b

    def ring_analysis(self, f):
        """[c, npix] -> S and D = G_N +- G_S, [lmax + 1, ring, 2 c] (real parts, then imaginary)."""
        c = f.shape[0]
        S = torch.empty((self.lmax + 1, self.q, 2 * c), dtype=torch.float64, device="cuda")
        D = torch.empty_like(S)
        for (n, ph), rs in self._ring_sets().items():
            co, si = self._phases(n, ph)
            a, b = self._pixels(rs, n)
            gn = f[:, a].reshape(-1, n)
            gs = f[:, b].reshape(-1, n)
            if rs[-1] == self.q - 1:                         # the equator has no mirror ring
                gs = gs.view(c, len(rs), n).clone()
                gs[:, -1] = 0.0
                gs = gs.view(-1, n)
            for X, x in ((S, gn + gs), (D, gn - gs)):
                re = (x @ co).view(c, len(rs), -1).permute(2, 1, 0)
                im = (x @ si).view(c, len(rs), -1).permute(2, 1, 0)
                X[:, rs] = torch.cat([re, -im], 2)
        return S, D

    def ring_synthesis(self, E, O):
        """E and O [lmax + 1, 2 c, ring] -> [c, npix]."""
        c = E.shape[1] // 2
        out = torch.empty((c, 12 * self.nside ** 2), dtype=torch.float64, device="cuda")
        w = torch.full((self.lmax + 1, 1), 2.0, dtype=torch.float64, device="cuda")
        w[0] = 1.0
        for (n, ph), rs in self._ring_sets().items():
            co, si = self._phases(n, ph)
            co, si = (w * co.t()).contiguous(), (w * si.t()).contiguous()
            a, b = self._pixels(rs, n)
            for idx, F in ((a, E[:, :, rs] + O[:, :, rs]), (b, E[:, :, rs] - O[:, :, rs])):
                F = F.permute(1, 2, 0).contiguous()
                x = F[:c].reshape(c * len(rs), -1) @ co - F[c:].reshape(c * len(rs), -1) @ si
                x = x.view(c, len(rs), n)
                if idx is b and rs[-1] == self.q - 1:
                    idx, x = idx[:-1], x[:, :-1]
                out[:, idx] = x
        return out

    def _seeds(self, s):
        """Mantissa and exponent of the first nonzero function of each m (l = max(m, |s|)), [lmax + 1, ring]."""
        z = self.z_np.astype(np.longdouble)
        sh, ch = np.sqrt((1 - z) / 2), np.sqrt((1 + z) / 2)
        f = math.factorial
        man = np.zeros((self.lmax + 1, self.q))
        ex = np.zeros((self.lmax + 1, self.q), dtype=np.int64)
        a = abs(s)
        cur, e = None, np.zeros(self.q, dtype=np.int64)
        for m in range(self.lmax + 1):
            if m <= a:
                k = np.sqrt(np.longdouble((2 * a + 1) * f(2 * a)) / (f(a + m) * f(a - m)) / (4 * np.longdouble(np.pi)))
                k = -k if (m if s >= 0 else a) % 2 else k
                cur = k * (sh ** (a + m) * ch ** (a - m) if s >= 0 else sh ** (a - m) * ch ** (a + m))
            else:
                r = np.sqrt(np.longdouble((2 * m + 1) * (2 * m)) / ((m + s) * (m - s)))
                cur = -r * sh * ch * cur
            cur, d = np.frexp(cur)
            e = (0 if m <= a else e) + d.astype(np.int64)
            man[m], ex[m] = cur, e
        return man, ex

    def functions(self, s):
        """Yields (i0, L) with L [m <= lmax - i0, STEPS, ring] = s_lambda_{m+i, m} for i0 <= i < i0 + STEPS, in
        64 bits; values far below 2^-400 of the others come out as zero. Rows past lmax are zero."""
        lm, a = self.lmax, abs(s)
        man, ex = self._seeds(s)
        k = np.maximum(0, -((ex + 400) // 512))             # carried as value = v 2^(-512 k)
        v0 = torch.from_numpy(np.ldexp(man, (ex + 512 * k).astype(np.int32))).cuda()
        k = torch.from_numpy(k).cuda()
        mm = np.arange(lm + 1, dtype=np.longdouble)
        first = torch.from_numpy(np.maximum(a - np.arange(lm + 1), 0)).cuda()
        y1, y0 = torch.zeros_like(v0), torch.zeros_like(v0)
        on = (k == 0).double()
        for i0 in range(0, lm + 1, self.STEPS):
            M = lm + 1 - i0
            y1, y0, on, k, v0, first = y1[:M], y0[:M], on[:M], k[:M], v0[:M], first[:M]
            out = torch.zeros((M, self.STEPS, self.q), dtype=torch.float64, device="cuda")
            for i in range(i0, min(i0 + self.STEPS, lm + 1)):
                m = mm[:M]
                l = m + i - 1                                # y_{l+1} = (A z + B) y_l - C y_{l-1}
                with np.errstate(all="ignore"):
                    K = np.sqrt(((l + 1) ** 2 - m * m) * ((l + 1) ** 2 - s * s))
                    w = np.sqrt((2 * l + 3) * (2 * l + 1))
                    A = w * (l + 1) / K
                    B = w * m * s / (l * K) if s else 0 * l
                    C = (l + 1) * np.sqrt((2 * l + 3) * (l * l - m * m) * (l * l - s * s)) / (
                        np.where(l > 0, l, 1) * np.sqrt(np.maximum(2 * l - 1, 1)) * K)
                live = (m + i > np.maximum(m, a))
                A, B, C = (torch.from_numpy(np.where(live, x, 0).astype(np.float64)).cuda()[:, None] for x in (A, B, C))
                y = (A * self.z + B) * y1 - C * y0
                here = (first == i)
                if i <= a:
                    y = torch.where(here[:, None], v0, y)
                y0, y1 = y1, y
                out[:, i - i0] = y * on
                if i % 4 == 3:
                    big = (k > 0) & (torch.maximum(y0.abs(), y1.abs()) > 2.0 ** 64)
                    f = torch.where(big, torch.full_like(y0, 2.0 ** -512), torch.ones_like(y0))
                    y0, y1 = y0 * f, y1 * f
                    k = k - big.long()
                    on = (k == 0).double()
            for j in range(self.STEPS):                      # rows of m with m + i > lmax
                out[max(0, lm + 1 - i0 - j):, j] = 0.0
            yield i0, out

    def index(self, i):
        """Packed positions of l = m + i, m = 0 .. lmax - i."""
        m = torch.arange(self.lmax + 1 - i, device="cuda")
        return m * (2 * self.lmax + 1 - m) // 2 + m + i

    def analysis(self, f, scale=1.0):
        """[c, npix] -> alm [c, N_lm]."""
        c = f.shape[0]
        S, D = self.ring_analysis(f)
        out = torch.zeros((c, (self.lmax + 1) * (self.lmax + 2) // 2), dtype=torch.complex128, device="cuda")
        for i0, L in self.functions(0):
            M = L.shape[0]
            for par, X in ((0, S), (1, D)):
                a = torch.bmm(L[:, par::2].contiguous(), X[:M])   # i0 is even
                for h in range(a.shape[1]):
                    i = i0 + 2 * h + par
                    if i <= self.lmax:
                        v = a[:self.lmax + 1 - i, h] * (self.omega * scale)
                        out[:, self.index(i)] = torch.complex(v[:, :c], v[:, c:]).t()
        return out

    def synthesis(self, alm):
        """alm [c, N_lm] -> [c, npix]."""
        c = alm.shape[0]
        E = torch.zeros((self.lmax + 1, 2 * c, self.q), dtype=torch.float64, device="cuda")
        O = torch.zeros_like(E)
        for i0, L in self.functions(0):
            M = L.shape[0]
            for par, X in ((0, E), (1, O)):
                X[:M] += torch.bmm(self.columns(alm, i0 + par, M), L[:, par::2].contiguous())
        return self.ring_synthesis(E, O)

    def columns(self, alm, i, M):
        """[M, 2 c, STEPS / 2]: alm of l = m + i, m + i + 2, ... (real parts, then imaginary; real at m = 0)."""
        c = alm.shape[0]
        b = torch.zeros((M, 2 * c, self.STEPS // 2), dtype=torch.float64, device="cuda")
        for h in range(self.STEPS // 2):
            if i + 2 * h <= self.lmax:
                v = alm[:, self.index(i + 2 * h)]
                b[:v.shape[1], :c, h] = v.real.t()
                b[:v.shape[1], c:, h] = v.imag.t()
        b[0, c:] = 0.0
        return b

    # E and B: with lambda+- = ((2)lambda +- (-2)lambda) / 2, whose parities under z -> -z are (-1)^(l+m) and the
    # opposite, E = -sum (lambda+ Q + i lambda- U), B = sum (-lambda+ U + i lambda- Q); Q, U the adjoint
    def pol_analysis(self, q, u):
        out = torch.zeros((2, (self.lmax + 1) * (self.lmax + 2) // 2), dtype=torch.complex128, device="cuda")
        S, D = self.ring_analysis(torch.stack([q, u]))
        for (i0, P), (_, N) in zip(self.functions(2), self.functions(-2)):
            plus, minus = 0.5 * (P + N), 0.5 * (P - N)
            M = P.shape[0]
            for par in (0, 1):
                X, Y = (S, D) if par == 0 else (D, S)
                a = torch.bmm(plus[:, par::2].contiguous(), X[:M])
                b = torch.bmm(minus[:, par::2].contiguous(), Y[:M])
                for h in range(a.shape[1]):
                    i = i0 + 2 * h + par
                    if i <= self.lmax:
                        n = self.lmax + 1 - i
                        pq, pu = torch.complex(a[:n, h, 0], a[:n, h, 2]), torch.complex(a[:n, h, 1], a[:n, h, 3])
                        mq, mu = torch.complex(b[:n, h, 0], b[:n, h, 2]), torch.complex(b[:n, h, 1], b[:n, h, 3])
                        out[0, self.index(i)] = -self.omega * (pq + 1j * mu)
                        out[1, self.index(i)] = self.omega * (-pu + 1j * mq)
        return out

    def pol_synthesis(self, e, b):
        alm = torch.stack([e, b]).clone()
        alm[:, :self.lmax + 1] = alm[:, :self.lmax + 1].real + 0j
        E = torch.zeros((self.lmax + 1, 4, self.q), dtype=torch.float64, device="cuda")
        O = torch.zeros_like(E)
        plus_in = -alm                                       # Q += lambda+ (-E), U += lambda+ (-B)
        minus_in = torch.stack([-1j * alm[1], 1j * alm[0]])   # Q += lambda- (-i B), U += lambda- (i E)
        for (i0, P), (_, N) in zip(self.functions(2), self.functions(-2)):
            plus, minus = 0.5 * (P + N), 0.5 * (P - N)
            M = P.shape[0]
            for par in (0, 1):
                X, Y = (E, O) if par == 0 else (O, E)
                X[:M] += torch.bmm(self._all(plus_in, i0 + par, M), plus[:, par::2].contiguous())
                Y[:M] += torch.bmm(self._all(minus_in, i0 + par, M), minus[:, par::2].contiguous())
        f = self.ring_synthesis(E, O)
        return f[0], f[1]

    def _all(self, alm, i, M):
        b = torch.zeros((M, 4, self.STEPS // 2), dtype=torch.float64, device="cuda")
        for h in range(self.STEPS // 2):
            if i + 2 * h <= self.lmax:
                v = alm[:, self.index(i + 2 * h)]
                b[:v.shape[1], :2, h] = v.real.t()
                b[:v.shape[1], 2:, h] = v.imag.t()
        return b


def _filtered(alm, cl, x, lmax):
    """C_l / (C_l + x) alm, zero where C_l is."""
    f = np.where(cl > 0, cl / np.where(cl > 0, cl + x, 1.0), 0.0)
    return alm * torch.from_numpy(f[_packed(lmax)[1]]).cuda()


def _solve(nside, lmax, cl, ninv, d, lams, bands=None):
    """Sweeps of Eqs. (3) and (4) from s = 0: (map, alm) of the last iterate."""
    d = d.double()
    q = ninv / ninv.max()
    tau = 1.0 / float(ninv.max())
    s = torch.zeros_like(d)
    for k, lam in enumerate(lams):
        L = lmax if bands is None else int(bands[k])
        if k == 0 or sph.lmax != L:
            sph = _Sphere(nside, L)
        t = s + lam * q / (1.0 + (lam - 1.0) * q) * (d - s)
        alm = _filtered(sph.analysis(t), cl[:L + 1], lam * tau * sph.omega, L)
        s = sph.synthesis(alm)
    return s, alm


def _pol_solve(nside, lmax, cl4, ninv6, bits, d, lams):
    """The polarised sweeps (T uncorrelated with Q and U in the noise)."""
    ot, op = (bits & 1).double(), ((bits >> 1) & 1).double()
    a, b, c, x = ninv6[0] * ot, ninv6[1] * op, ninv6[2] * op, ninv6[5] * op
    eig = 0.5 * (b + c) + torch.sqrt(0.25 * (b - c) ** 2 + x * x)
    tau = 1.0 / float(torch.maximum(a, eig).max())
    a, b, c, x = a * tau, b * tau, c * tau, x * tau
    sph = _Sphere(nside, lmax)
    l = _packed(lmax)[1]
    tt, ee, bb, te = (torch.from_numpy(v[l]).cuda() for v in cl4)
    s = torch.zeros_like(d)
    for lam in lams:
        r = d - s
        t = torch.empty_like(d)
        t[0] = s[0] + lam * a / (1.0 + (lam - 1.0) * a) * r[0]
        v1, v2 = b * r[1] + x * r[2], x * r[1] + c * r[2]
        n11, n22, n12 = 1.0 + (lam - 1.0) * b, 1.0 + (lam - 1.0) * c, (lam - 1.0) * x
        det = n11 * n22 - n12 * n12
        t[1] = s[1] + lam * (n22 * v1 - n12 * v2) / det
        t[2] = s[2] + lam * (n11 * v2 - n12 * v1) / det
        at = sph.analysis(t[:1])[0]
        ae, ab = sph.pol_analysis(t[1], t[2])
        mu = lam * tau * sph.omega
        de = tt * ee - te * te
        den = de + mu * (tt + ee) + mu * mu
        alm = torch.stack([((de + tt * mu) * at + te * mu * ae) / den, (te * mu * at + (de + ee * mu) * ae) / den,
                           bb / (bb + mu) * ab])
        s = torch.stack([sph.synthesis(alm[:1])[0], *sph.pol_synthesis(alm[1], alm[2])])
    return s, alm


def exact(case, seed):
    kind, nside, lmax, maps = case["kind"], case["nside"], case["lmax"], case["maps"]
    rt = _real(case["dtype"])
    lams = _schedule(case.get("sweeps", 1))
    # about 0.7 s a transform at lmax 1024, twice that with polarisation, which goes map by map
    if 1.4 * len(lams) * lmax / 1024.0 * (2.0 * maps if kind == "pol" else 1.0) > 20.0:
        return None
    if kind == "pol":
        cl4, ninv6, bits, d = _pol_problem(nside, lmax, maps, seed)
        r = [_pol_solve(nside, lmax, cl4, ninv6, bits, d[i], lams) for i in range(maps)]
        s, a = torch.stack([x[0] for x in r]), torch.stack([x[1] for x in r])
        return (s, a) if maps > 1 else (s[0], a[0])
    if kind == "group":
        r = []
        for k, (n, ns, lm) in enumerate(GROUP):
            cl, ninv, d = _problem(ns, lm, n, 31 * seed + k, rt)
            r.append(_solve(ns, lm, cl, ninv, d, lams))
        return [x[0] for x in r], [x[1] for x in r]
    if kind == "served":
        r = []
        for k, ns in enumerate(SERVED):
            cl, ninv, d = _request(k, ns, seed)
            r.append(_solve(ns, 2 * ns, cl, ninv, d[None], lams)[0][0])
        return r
    cl, ninv, d = _problem(nside, lmax, maps, seed, rt)
    if kind in ("synthesis", "pair"):
        a = _alm(lmax, maps, seed, rt, cl).to(torch.complex128)
    sph = _Sphere(nside, lmax)
    if kind == "analysis":
        r = (sph.analysis(d.double()),)
    elif kind == "synthesis":
        r = (sph.synthesis(a),)
    elif kind == "pair":
        # the analysed map is the synthesised one
        m = sph.synthesis(a)
        r = (m, sph.analysis(m))
    else:
        bands = _bands(lmax, case["sweeps"]) if kind == "banded" else None
        r = _solve(nside, lmax, cl, ninv, d, lams, bands)
        if bands is not None and r[1].shape[1] != (lmax + 1) * (lmax + 2) // 2:
            # the last sweeps of a short schedule may be truncated too: zero above their band
            L = int(bands[-1])
            m, l = _packed(lmax)
            full = torch.zeros((1, len(l)), dtype=torch.complex128, device="cuda")
            full[:, torch.from_numpy(np.nonzero(l <= L)[0]).cuda()] = r[1]
            r = (r[0], full)
    r = tuple(x if maps > 1 else x[0] for x in r)
    return r[0] if len(r) == 1 else r
