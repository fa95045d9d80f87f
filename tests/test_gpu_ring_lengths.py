"""Ring stages at the lengths where the transform's form changes: the class
lengths themselves (compile-time stages), Bluestein of a ring pair and of single
rings as half-length complex transforms in every class, at their shortest and
longest lengths, and the folds (one term per bin, columns of very short rings,
aliases), with both Delta layouts, against the oracle's plain DFTs.

Tolerance: 1e-12 relative RMS per ring, the bar of every FP64 result; a
transform of 8192 points and Bluestein's two contribute a few 1e-15."""
import numpy as np
import pytest

import oracle
import sht_inputs as si

pytestmark = pytest.mark.gpu
TOL = 1e-12

# class lengths; pairs under Bluestein (odd); halves (even); direct; very short
LENGTHS = [1024, 2048, 4096, 8192, 509, 1021, 2049, 4093, 4097, 1018, 1042, 2042, 2062, 4082, 4098, 4106, 8186,
           8182, 4095, 2044, 4, 12, 28, 100, 255, 256, 257, 260, 508]


def say(msg):
    print(f"[gpu] {msg}", flush=True)


def relrms(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def rings(nphi, seed, phi0=None):
    rng = np.random.default_rng(seed)
    nr = len(nphi)
    th = np.sort(rng.uniform(0.05, 3.09, nr))
    p0 = rng.uniform(-1.0, 2.0, nr) if phi0 is None else np.full(nr, phi0)
    return si._pack(th, np.array(nphi, dtype=np.int32), p0, rng.uniform(0.2, 1.0, nr), f"lengths{seed}")


@pytest.mark.parametrize("mmax", [7, 600, 2048, 4096])
@pytest.mark.parametrize("twice", [False, True])
def test_ring_lengths(mmax, twice):
    """Each length once and twice (a pair of one phase, or two phases), a
    phase of zero in the second case."""
    import torch
    import paper_1106_0159_amd as sht
    lens = LENGTHS if mmax < 4096 else [n for n in LENGTHS if n > 500 or n == 28]
    g = rings(np.repeat(lens, 2) if twice else lens, 50 + mmax, 0.0 if twice and mmax == 2048 else None)
    rng = np.random.default_rng(mmax)
    d = rng.standard_normal((g.nrings, mmax + 1)) + 1j * rng.standard_normal((g.nrings, mmax + 1))
    s = si.random_map(g, mmax)
    say(f"ring lengths mmax={mmax} twice={twice}")
    got = sht.delta2map(torch.from_numpy(d).cuda(), g, mmax).cpu().numpy()
    gotd = sht.map2delta(torch.from_numpy(s).cuda(), g, mmax).cpu().numpy()
    ref, refd = oracle.delta2map(mmax, g, d), oracle.map2delta(mmax, g, s)
    for r in range(g.nrings):
        o, n = int(g.ofs[r]), int(g.nphi[r])
        assert relrms(got[o:o + n], ref[o:o + n]) <= TOL, (n, relrms(got[o:o + n], ref[o:o + n]))
        assert relrms(gotd[r], refd[r]) <= TOL, (n, relrms(gotd[r], refd[r]))


@pytest.mark.parametrize("nmaps", [1, 2, 7, 9])
def test_ring_lengths_map_minor(nmaps):
    """Map-minor Delta: the same values as ring-major."""
    import torch
    import paper_1106_0159_amd as sht
    mmax, X = 700, sht.SHT_DELTA_MAP_MINOR
    g = rings(LENGTHS, 3)
    rng = np.random.default_rng(nmaps)
    d = rng.standard_normal((nmaps, g.nrings, mmax + 1)) + 1j * rng.standard_normal((nmaps, g.nrings, mmax + 1))
    s = np.stack([si.random_map(g, 5 + k) for k in range(nmaps)])
    say(f"ring lengths, map-minor, {nmaps} maps")
    dm = torch.from_numpy(np.ascontiguousarray(np.moveaxis(d, 0, 2))).cuda()
    got = sht.delta2map(dm, g, mmax, flags=X).cpu().numpy()
    gotd = np.moveaxis(sht.map2delta(torch.from_numpy(s).cuda(), g, mmax, flags=X).cpu().numpy(), 2, 0)
    for k in range(nmaps):
        assert relrms(got[k], oracle.delta2map(mmax, g, d[k])) <= TOL
        assert relrms(gotd[k], oracle.map2delta(mmax, g, s[k])) <= TOL
