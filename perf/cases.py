"""Performance cases of the spherical harmonic transforms.

A case is a transform call (or an uneven batch) as a user's program makes it:
the geometry handle, the plan, the workspace and the output buffer are kept by
the program, and one pass is one call through the public entry points of
paper_1106_0159_amd.  The cases cover both directions, both grids (HEALPix and
Gauss-Legendre), one map and batches of maps, FP64 and the mixed-precision
mode, and sizes from a launch-bound lmax of 64 to the serving mix's largest
lmax of 4096.
"""
import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1106_0159_amd as sht

MIXED_SYN = sht.SHT_MIXED | sht.SHT_MIXED_SPLIT_BF16  # the batched mode's synthesis; analysis takes SHT_MIXED


def _single(name, op, grid, n, nphi, lmax, mmax, nmaps, mixed=False):
    c = {"op": op, "grid": grid, "n": n, "nphi": nphi, "lmax": lmax, "mmax": mmax, "nmaps": nmaps, "mixed": mixed}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # the smallest request of the serving mix: latency and launches
        _single("ana_hp32_l64", "map2alm", "healpix", 32, 0, 64, 64, 1),
        # a small exact-quadrature synthesis, called back to back
        _single("syn_gl257_l256", "alm2map", "gl", 257, 513, 256, 256, 1),
        # ordinary odd-sized requests of the serving mix: N_side prime (polar
        # and belt rings of every factorisation) ...
        _single("syn_hp347_l694", "alm2map", "healpix", 347, 0, 694, 694, 1),
        # ... and a band-limited analysis with mmax < lmax on 17 * 53 points
        _single("ana_gl451_l450_m300", "map2alm", "gl", 451, 901, 450, 300, 1),
        # a few maps at once (intensity and polarisation components taken as
        # scalars, detector splits): FP64, below the mixed mode's batch size
        _single("syn_hp512_l1024_x4", "alm2map", "healpix", 512, 0, 1024, 1024, 4),
        # the benchmark's one map there ...
        _single("syn_hp1024_l2048", "alm2map", "healpix", 1024, 0, 2048, 2048, 1),
        # ... and back
        _single("ana_hp1024_l2048", "map2alm", "healpix", 1024, 0, 2048, 2048, 1),
        # the upper end of the serving mix
        _single("syn_hp2048_l4096", "alm2map", "healpix", 2048, 0, 4096, 4096, 1),
        # simulations: FP64 analysis of a batch on the exact grid of lmax 1024
        _single("ana_gl1025_l1024_x64", "map2alm", "gl", 1025, 2049, 1024, 1024, 64),
        # the batched mixed-precision mode, one direction each
        _single("syn_mixed_hp1024_l2048_x64", "alm2map", "healpix", 1024, 0, 2048, 2048, 64, True),
        _single("ana_mixed_hp1024_l2048_x32", "map2alm", "healpix", 1024, 0, 2048, 2048, 32, True),
        # an uneven batch: requests of many sizes, both directions, one launch
        {"name": "uneven_batch_64", "op": "batch", "requests": 64, "lmin": 128, "lmax": 2048, "trace": 4},
    ]


def _cost(lmax, mmax, nmaps, mixed):
    """Rough relative cost, to keep drawn cases below the largest listed one."""
    return lmax * lmax * mmax * nmaps * (0.3 if mixed else 1.0)


def draw(rng):
    """One more case: direction, grid, size (log-uniform) and batch drawn at random."""
    kind = rng.choice(["one", "one", "one", "few", "many", "mixed", "batch"])
    if kind == "batch":
        return {"op": "batch", "requests": rng.randint(8, 64), "lmin": 128,
                "lmax": int(round(math.exp(rng.uniform(math.log(256), math.log(2048))))),
                "trace": rng.randrange(1 << 16)}
    nmaps = {"one": 1, "few": rng.randint(2, 7),
             "many": int(round(math.exp(rng.uniform(math.log(8), math.log(64))))),
             "mixed": int(round(math.exp(rng.uniform(math.log(8), math.log(64)))))}[kind]
    mixed = kind == "mixed"
    op = rng.choice(["alm2map", "map2alm"])
    hi = 4096
    while True:
        lmax = int(round(math.exp(rng.uniform(math.log(64), math.log(hi)))))
        mmax = lmax if rng.random() < 0.8 else rng.randint(lmax // 4, lmax)
        if _cost(lmax, mmax, nmaps, mixed) <= 0.75 * _cost(2048, 2048, 64, True):
            break
    if rng.random() < 0.5:
        # N_side = lmax / 2 (the serving mix), now and then coarser or finer
        nside = max(8, min(2048, round(lmax / rng.choice([2, 2, 2, 1.5, 2.5]))))
        return _single(None, op, "healpix", nside, 0, lmax, mmax, nmaps, mixed)
    lmax = min(lmax, 3500)
    mmax = min(mmax, lmax)
    n = lmax + 1 + rng.choice([0, 0, rng.randint(1, 40)])
    return _single(None, op, "gl", n, 2 * mmax + 1 + rng.choice([0, 0, rng.randint(1, 100)]), lmax, mmax, nmaps, mixed)


# ---------------------------------------------------------------- geometry
_PI_L = np.longdouble("3.14159265358979323846264338327950288")


def _mirror(theta):
    return (_PI_L - theta.astype(np.longdouble)).astype(np.float64)


@functools.lru_cache(maxsize=None)
def _healpix(nside):
    """HEALPix rings (Gorski et al. 2005): caps of 4 i pixels, belt of 4 N_side."""
    i = np.arange(1, 2 * nside + 1)
    cap = i < nside
    theta = np.where(cap, 2.0 * np.arcsin(np.minimum(i / (math.sqrt(6.0) * nside), 1.0)),
                     np.arccos(np.minimum((4 * nside - 2 * i) / (3.0 * nside), 1.0)))
    nphi = np.where(cap, 4 * i, 4 * nside)
    phi0 = np.where(cap, np.pi / (4 * i), np.pi / (2 * nside) * (1.0 - 0.5 * ((i - nside + 1) % 2)))
    nr = 4 * nside - 1
    return _rings(np.concatenate([theta, _mirror(theta[:-1])[::-1]]), np.concatenate([nphi, nphi[:-1][::-1]]),
                  np.concatenate([phi0, phi0[:-1][::-1]]), np.full(nr, np.pi / (3.0 * nside * nside)))


@functools.lru_cache(maxsize=None)
def _gauss_legendre(n, nphi):
    """n Gauss-Legendre rings of nphi pixels, nodes by Newton iteration."""
    half = n // 2
    x = np.cos(np.pi * (np.arange(1, half + 1) - 0.25) / (n + 0.5)).astype(np.longdouble)
    for _ in range(4):
        p0, p1 = np.ones_like(x), x
        for k in range(2, n + 1):
            p0, p1 = p1, ((2 * k - 1) * x * p1 - (k - 1) * p0) / k
        dp = n * (x * p1 - p0) / (x * x - 1)
        x = x - p1 / dp
    w = (2 / ((1 - x * x) * dp * dp)).astype(np.float64)
    theta = np.arccos(x).astype(np.float64)
    mid = [2.0 - 2.0 * w.sum()] if n % 2 else []
    return _rings(np.concatenate([theta, [np.pi / 2] * (n % 2), _mirror(theta)[::-1]]), np.full(n, nphi),
                  np.zeros(n), np.concatenate([w, mid, w[::-1]]) * (2 * np.pi / nphi))


def _rings(theta, nphi, phi0, weight):
    nphi = nphi.astype(np.int32)
    ofs = np.concatenate([[0], np.cumsum(nphi[:-1], dtype=np.int64)])
    return SimpleNamespace(theta=np.ascontiguousarray(theta), nphi=nphi, phi0=np.ascontiguousarray(phi0, dtype=np.float64),
                           weight=np.ascontiguousarray(weight), ofs=ofs)


def _geometry(c):
    return _healpix(c["n"]) if c["grid"] == "healpix" else _gauss_legendre(c["n"], c["nphi"])


def _npix(g):
    return int(g.nphi.sum(dtype=np.int64))


def _trace(c):
    """The requests of an uneven batch: lmax log-uniform, each on its own grid."""
    rng = np.random.default_rng(1106 + c["trace"])
    out = []
    for k in range(c["requests"]):
        lmax = int(round(math.exp(rng.uniform(math.log(c["lmin"]), math.log(c["lmax"])))))
        op = "alm2map" if rng.random() < 0.5 else "map2alm"
        if k % 4 == 3:
            out.append(_single(None, op, "healpix", (lmax + 1) // 2, 0, lmax, lmax, 1))
        else:
            out.append(_single(None, op, "gl", lmax + 1, 2 * lmax + 1, lmax, lmax, 1))
    return out


# ---------------------------------------------------------------- inputs
@functools.lru_cache(maxsize=4)
def _spectrum(lmax, mmax):
    """Standard deviations of Re a_lm and Im a_lm, [nalm, 2]: C_l = 1/(l(l+1))
    for l >= 2, a_l0 real (m-major packed, as the transforms take a_lm)."""
    sd = np.zeros((sht.nalm(lmax, mmax), 2))
    cl = np.zeros(lmax + 1)
    l = np.arange(2, lmax + 1)
    cl[2:] = 1.0 / (l * (l + 1.0))
    for m in range(mmax + 1):
        at = m * (2 * lmax + 1 - m) // 2
        sd[at + m: at + lmax + 1] = np.sqrt(cl[m:] / 2)[:, None] if m else np.stack([np.sqrt(cl), 0 * cl], 1)
    return torch.from_numpy(sd).cuda()


def _input(c, seed):
    """Power-law a_lm (synthesis) or maps of white noise over a smooth sky (analysis)."""
    gen = torch.Generator("cuda").manual_seed(seed)
    if c["op"] == "alm2map":
        sd = _spectrum(c["lmax"], c["mmax"])
        a = torch.randn((c["nmaps"],) + tuple(sd.shape), dtype=torch.float64, device="cuda", generator=gen)
        return torch.view_as_complex(a.mul_(sd))
    g = _geometry(c)
    s = torch.randn((c["nmaps"], _npix(g)), dtype=torch.float64, device="cuda", generator=gen)
    t = torch.from_numpy(np.repeat(np.cos(g.theta), g.nphi)).cuda()
    amp = torch.randn((c["nmaps"], 3), dtype=torch.float64, device="cuda", generator=gen)
    for k in range(3):
        s.addcmul_(t ** k, amp[:, k:k + 1])
    return s


def prepare(case, seed):
    if case["op"] == "batch":
        reqs = _trace(case)
        sht.plan_cache_limits(max(8, 2 * len(reqs)), max(32, 2 * len(reqs)))
        handles = [sht.GeomHandle(_geometry(r)) for r in reqs]
        ins = [_input(r, seed + 1000003 * k)[0] for k, r in enumerate(reqs)]
        batch = sht.Batch([(r["op"], r["lmax"], h, x, None) for r, h, x in zip(reqs, handles, ins)])
        return SimpleNamespace(op="batch", batch=batch, inputs=ins)
    h = sht.GeomHandle(_geometry(case))
    flags = 0 if not case["mixed"] else MIXED_SYN if case["op"] == "alm2map" else sht.SHT_MIXED
    lmax, mmax, nmaps = case["lmax"], case["mmax"], case["nmaps"]
    sht.prepare(h, lmax, mmax)
    x = _input(case, seed)
    ws = sht.workspace(lmax, mmax, h, nmaps, "cuda", flags)
    if case["op"] == "alm2map":
        out = torch.empty((nmaps, h.npix), dtype=torch.float64, device="cuda")
    else:
        out = torch.empty((nmaps, sht.nalm(lmax, mmax)), dtype=torch.complex128, device="cuda")
    return SimpleNamespace(op=case["op"], geom=h, lmax=lmax, mmax=mmax, flags=flags, x=x, out=out, ws=ws)


def run(state):
    if state.op == "batch":
        state.batch.run()
        return list(state.batch.outputs)
    f = sht.alm2map if state.op == "alm2map" else sht.map2alm
    return f(state.x, state.geom, state.lmax, state.mmax, out=state.out, ws=state.ws, flags=state.flags)


# ---------------------------------------------------------------- work
@functools.lru_cache(maxsize=None)
def _terms(grid, n, nphi, lmax, mmax):
    """Terms (ring pair, l, m) that are not exponentially small (l sin theta >= m),
    and the flops of the ring FFTs of one map (2.5 N log2 N per real ring)."""
    g = _healpix(n) if grid == "healpix" else _gauss_legendre(n, nphi)
    s = np.sin(g.theta[: (len(g.theta) + 1) // 2])
    m = np.arange(mmax + 1)
    terms = sum(int(np.maximum(0, lmax + 1 - np.maximum(m, np.ceil(m / sr))).sum()) for sr in s)
    nf = g.nphi.astype(np.float64)
    return terms, float((2.5 * nf * np.log2(np.maximum(nf, 2))).sum())


def work(case):
    if case["op"] == "batch":
        parts = [work(r) for r in _trace(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    terms, fft = _terms(case["grid"], case["n"], case["nphi"], case["lmax"], case["mmax"])
    nmaps = case["nmaps"]
    nbytes = nmaps * (8 * _npix(_geometry(case)) + 16 * sht.nalm(case["lmax"], case["mmax"]))
    # per term the recurrence (4 flops, once for all maps) and a complex by
    # real multiply-add (4 flops) per map
    return {"bytes": nbytes, "flops": terms * (4 + 4 * nmaps) + nmaps * fft}


# ---------------------------------------------------------------- 64-bit reference
def _split(v):
    """A long double array as head (26 bits, so that products of two heads are
    exact) and rest, in FP64 on the GPU."""
    f = v.astype(np.float64) * 134217729.0  # 2^27 + 1
    head = f - (f - v.astype(np.float64))
    return torch.from_numpy(head).cuda(), torch.from_numpy((v - head).astype(np.float64)).cuda()


def _legendre_blocks(theta, lmax, mmax, values):
    """Blocks of normalised lambda_lm(cos theta) for m >= 0: yields (m0, l0,
    lam[l, m, ring]) over all l >= m0 (zero for l < m), at most `values` values
    at a time.  The recurrence of Sec. 2.2 with an exponent per (m, ring); the
    coefficients and cos theta are carried to more than FP64 (head and rest),
    since their rounding would add up along l more than that of the values."""
    th = theta.astype(np.longdouble)
    xh, xr = (v[None, :] for v in _split(np.cos(th)))
    s = np.sin(th)[None, :]
    mu = np.empty(mmax + 1, dtype=np.longdouble)
    mu[0] = 1 / np.sqrt(4 * _PI_L)
    for m in range(1, mmax + 1):
        mu[m] = -mu[m - 1] * np.sqrt(np.longdouble(2 * m + 1) / (2 * m))
    nm = max(1, min(mmax + 1, (1 << 19) // theta.size))
    for m0 in range(0, mmax + 1, nm):
        ms = np.arange(m0, min(mmax + 1, m0 + nm))
        man, ex = np.frexp(mu[ms][:, None] * s ** ms[:, None].astype(np.longdouble))
        sc = -np.maximum(0, (-ex.astype(np.int64) - 100) // 600)  # value = carrier * 2^(600 sc)
        carrier = np.ldexp(man.astype(np.float64), np.clip(ex - 600 * sc, -1000, 1000).astype(np.int32))
        carrier[man == 0] = 0.0
        seed, sc = torch.from_numpy(carrier).cuda(), torch.from_numpy(sc).cuda()
        p1, p2 = torch.zeros_like(seed), torch.zeros_like(seed)
        ls = np.arange(m0, lmax + 1, dtype=np.longdouble)[:, None]
        mm = ms.astype(np.longdouble)[None, :]
        with np.errstate(all="ignore"):
            beta = np.where(ls > mm, np.sqrt((4 * ls * ls - 1) / (ls * ls - mm * mm)), 0)
            ratio = np.where(ls > mm + 1, beta / np.sqrt((4 * (ls - 1) ** 2 - 1) / ((ls - 1) ** 2 - mm * mm)), 0)
        (bh, br), (rh, rr) = ((h[:, :, None], r[:, :, None]) for h, r in (_split(beta), _split(ratio)))
        nl = max(1, values // (len(ms) * theta.size))
        for l0 in range(m0, lmax + 1, nl):
            lam = torch.empty((min(nl, lmax + 1 - l0), len(ms), theta.size), dtype=torch.float64, device="cuda")
            for i in range(lam.shape[0]):
                k = l0 + i - m0
                # beta x p1 - ratio p2, the exact product of the heads first
                e = (bh[k] * xr).addcmul_(br[k], xh).addcmul_(br[k], xr).mul_(p1).addcmul_(rr[k], p2, value=-1)
                p = e.addcmul_(bh[k] * xh, p1).addcmul_(rh[k], p2, value=-1)
                if k < len(ms):
                    p[k] = seed[k]
                p1, p2 = p, p1
                if i % 16 == 15 or i == lam.shape[0] - 1:
                    big = (sc < 0) & (p1.abs() > 2.0 ** -60)
                    p1, p2, sc = torch.where(big, p1 * 2.0 ** -600, p1), torch.where(big, p2 * 2.0 ** -600, p2), sc + big
                lam[i] = torch.where(sc == 0, p1, 0.0)
            yield m0, l0, lam


def _columns(lmax, m0, nm, l0, nl):
    """Packed positions of the block a[l, m], and where l >= m."""
    l = torch.arange(l0, l0 + nl, device="cuda")[:, None]
    m = torch.arange(m0, m0 + nm, device="cuda")[None, :]
    at = (m * (2 * lmax + 1 - m) // 2 + l).clamp(min=0)
    return at, l >= m


def _dft_rows(g, r, mmax):
    """e^{i m phi_j} of ring r as cos and sin, [mmax + 1, nphi], angles reduced exactly."""
    n = int(g.nphi[r])
    m = torch.arange(mmax + 1, device="cuda")
    j = torch.arange(n, device="cuda")
    a = (m[:, None] * j[None, :] % n).double() * (2 * math.pi / n)
    p = torch.from_numpy(np.mod(np.arange(mmax + 1) * np.longdouble(g.phi0[r]), 2 * _PI_L).astype(np.float64)).cuda()
    a = a + p[:, None]
    return torch.cos(a), torch.sin(a)


def _ring_groups(g):
    """Rings of equal length and phase, which share one transform matrix."""
    groups = {}
    for r in range(len(g.theta)):
        groups.setdefault((int(g.nphi[r]), float(g.phi0[r])), []).append(r)
    return groups.values()


def _exact_one(c, x):
    """x: [nmaps, ...] inputs; the transform as plain sums in FP64."""
    g, lmax, mmax, nmaps = _geometry(c), c["lmax"], c["mmax"], c["nmaps"]
    nr, na = len(g.theta), sht.nalm(lmax, mmax)
    north = (nr + 1) // 2  # rings are mirror pairs r, nr - 1 - r about the equator
    xs = torch.view_as_real(x).contiguous() if x.is_complex() else x
    delta = torch.zeros((mmax + 1, nr, nmaps, 2), dtype=torch.float64, device="cuda")
    if c["op"] == "map2alm":
        for rings in _ring_groups(g):
            cs, sn = _dft_rows(g, rings[0], mmax)
            n = int(g.nphi[rings[0]])
            s = torch.stack([xs[:, g.ofs[r]:g.ofs[r] + n] * float(g.weight[r]) for r in rings]).reshape(-1, n)
            delta[:, rings, :, 0] = (cs @ s.T).reshape(mmax + 1, len(rings), nmaps)
            delta[:, rings, :, 1] = -(sn @ s.T).reshape(mmax + 1, len(rings), nmaps)
    out = torch.zeros((nmaps, na, 2), dtype=torch.float64, device="cuda")
    south = torch.arange(nr - 1, nr - 1 - north, -1, device="cuda")
    own = torch.arange(north, device="cuda") == south  # the equator ring counts once
    for m0, l0, lam in _legendre_blocks(g.theta[:north], lmax, mmax, 1 << 26):
        nl, nm = lam.shape[0], lam.shape[1]
        at, ok = _columns(lmax, m0, nm, l0, nl)
        for par in (0, 1):
            # l - m of this parity: the southern ring takes (-1)^(l+m) of the northern value
            sel = ok & ((torch.arange(l0, l0 + nl, device="cuda")[:, None]
                         + torch.arange(m0, m0 + nm, device="cuda")[None, :]) % 2 == par)
            lm = (lam * sel[:, :, None]).permute(1, 0, 2).contiguous()  # [m, l, ring]
            sign = 1.0 - 2.0 * par
            d = delta[m0:m0 + nm]
            if c["op"] == "alm2map":
                a = (xs[:, at] * sel[None, :, :, None]).permute(2, 1, 0, 3).reshape(nm, nl, -1).contiguous()
                v = torch.bmm(lm.transpose(1, 2).contiguous(), a).reshape(nm, north, nmaps, 2)
                d[:, :north] += v
                v[:, own] = 0.0
                d[:, south] += sign * v
            else:
                both = d[:, :north] + sign * d[:, south] * (~own)[None, :, None, None]
                v = torch.bmm(lm, both.reshape(nm, north, -1).contiguous()).reshape(nm, nl, nmaps, 2)
                pos = at[sel]
                out[:, pos] = v.permute(1, 0, 2, 3)[sel].permute(1, 0, 2)
    if c["op"] == "map2alm":
        out[:, : lmax + 1, 1] = 0.0
        return torch.view_as_complex(out)
    w = torch.full((mmax + 1, 1, 1), 2.0, dtype=torch.float64, device="cuda")
    w[0] = 1.0
    mp = torch.empty((nmaps, _npix(g)), dtype=torch.float64, device="cuda")
    delta[0, ..., 1] = 0.0
    for rings in _ring_groups(g):
        cs, sn = _dft_rows(g, rings[0], mmax)
        n = int(g.nphi[rings[0]])
        d = delta[:, rings] * w[..., None]
        s = d[..., 0].reshape(mmax + 1, -1).T.contiguous() @ cs - d[..., 1].reshape(mmax + 1, -1).T.contiguous() @ sn
        s = s.reshape(len(rings), nmaps, n)
        for k, r in enumerate(rings):
            mp[:, g.ofs[r]:g.ofs[r] + n] = s[k]
    return mp


def exact(case, seed):
    if case["op"] == "batch":
        # the small and middling requests (the sums of the largest would take too long)
        return [_exact_one(r, _input(r, seed + 1000003 * k))[0] if r["lmax"] <= 1200 else None
                for k, r in enumerate(_trace(case))]
    return _exact_one(case, _input(case, seed))
