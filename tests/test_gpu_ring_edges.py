"""Ring stages at edges that other tests leave out: Im Delta_0 that is not a
number, the lengths that meet Bluestein's shortest cyclic length, and odd lengths
above the largest Bluestein pair, whose direct prime stages a whole transform
runs through.

Tolerance: none where a value must be ignored; 1e-12 relative RMS per ring
against the oracle's plain DFTs, the bar of every FP64 result."""
import numpy as np
import pytest

import oracle
import sht_inputs as si

pytestmark = pytest.mark.gpu
TOL = 1e-12


def relrms(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def rings(nphi, seed, phi0=None):
    rng = np.random.default_rng(seed)
    nr = len(nphi)
    th = np.sort(rng.uniform(0.05, 3.09, nr))
    p0 = rng.uniform(-1.0, 2.0, nr) if phi0 is None else np.full(nr, phi0)
    return si._pack(th, np.array(nphi, dtype=np.int32), p0, rng.uniform(0.2, 1.0, nr), f"edges{seed}")


@pytest.mark.parametrize("phi0", [None, 0.3, 0.0])
@pytest.mark.parametrize("nmaps,minor", [(1, False), (2, False), (3, True)])
def test_imaginary_part_of_order_zero_is_ignored(phi0, nmaps, minor):
    """Im Delta_0 does not enter a map, also where it is infinite or NaN: every
    form of the fold (longer and shorter than mmax, single rings and pairs)."""
    import torch
    import paper_1106_0159_amd as sht
    mmax = 60
    g = rings(np.repeat([4, 28, 59, 61, 100, 120, 121, 256, 1018, 1024, 1026, 2049], 2), 7, phi0)
    rng = np.random.default_rng(8)
    d = rng.standard_normal((nmaps, g.nrings, mmax + 1)) + 1j * rng.standard_normal((nmaps, g.nrings, mmax + 1))
    d[:, :, 0] = d[:, :, 0].real
    bad = d.copy()
    bad.imag[:, :, 0] = np.resize([np.nan, np.inf, -np.inf, 1e300], g.nrings)
    flags = sht.SHT_DELTA_MAP_MINOR if minor else 0

    def run(x):
        x = np.ascontiguousarray(np.moveaxis(x, 0, 2)) if minor else x
        return sht.delta2map(torch.from_numpy(x).cuda(), g, mmax, flags=flags).cpu().numpy()

    print(f"[gpu] Im Delta_0: phi0 {phi0}, {nmaps} maps, map-minor {minor}", flush=True)
    assert np.array_equal(run(bad), run(d))


@pytest.mark.parametrize("mmax", [40, 700, 2600])
def test_shortest_bluestein_lengths(mmax):
    """Lengths whose cyclic convolution is exactly 2n - 2 points of a class, where
    the offsets +-(n-1) of the even chirp share one index: pairs of 2049 = 3 x 683
    and 4097 = 17 x 241 points, halves of 4098 (the shorter ones of that kind, 513,
    1025, 1026 and 2050, run as direct stages of 19 and 41 terms)."""
    import torch
    import paper_1106_0159_amd as sht
    g = rings(np.repeat([2049, 4097, 4098, 513, 1025, 1026, 2050], 2), 9 + mmax)
    rng = np.random.default_rng(mmax)
    d = rng.standard_normal((g.nrings, mmax + 1)) + 1j * rng.standard_normal((g.nrings, mmax + 1))
    s = si.random_map(g, mmax)
    print(f"[gpu] shortest Bluestein lengths mmax={mmax}", flush=True)
    got = sht.delta2map(torch.from_numpy(d).cuda(), g, mmax).cpu().numpy()
    back = sht.map2delta(torch.from_numpy(s).cuda(), g, mmax).cpu().numpy()
    ref, refd = oracle.delta2map(mmax, g, d), oracle.map2delta(mmax, g, s)
    for r in range(g.nrings):
        o, n = int(g.ofs[r]), int(g.nphi[r])
        assert relrms(got[o:o + n], ref[o:o + n]) <= TOL, (n, relrms(got[o:o + n], ref[o:o + n]))
        assert relrms(back[r], refd[r]) <= TOL, (n, relrms(back[r], refd[r]))


@pytest.mark.parametrize("nphi", [4101, 8173])
def test_whole_transform_with_direct_prime_stages(nphi):
    """Gauss-Legendre rings of 4101 = 3 x 1367 and 8173 = 11 x 743 points: odd and
    longer than the largest Bluestein pair, so that the whole transform runs
    through direct stages of 1367 and 743 terms, in both directions."""
    import torch
    import paper_1106_0159_amd as sht
    lmax = 300
    g = si.gauss_legendre(lmax + 1, nphi)
    a = si.powerlaw_alm(lmax, lmax, 11)
    s = si.random_map(g, 12)
    print(f"[gpu] whole transform, rings of {nphi}", flush=True)
    got = sht.alm2map(torch.from_numpy(a).cuda(), g, lmax).cpu().numpy()
    rs = np.arange(0, g.nrings, 10, dtype=np.int32)
    ref = oracle.alm2map(lmax, lmax, g, a, rings=rs)
    for r in rs:
        o = int(g.ofs[r])
        e = relrms(got[o:o + nphi], ref[o:o + nphi])
        assert e <= (TOL if r <= g.nrings // 2 else 1e-11), (int(r), e)  # the south by its mirror image
    back = sht.map2alm(torch.from_numpy(s).cuda(), g, lmax).cpu().numpy()
    ms = np.arange(0, lmax + 1, 10, dtype=np.int32)
    refa = oracle.map2alm(lmax, lmax, g, s, ms=ms)
    for m in ms:
        i = slice(si.alm_index(int(m), int(m), lmax), si.alm_index(lmax, int(m), lmax) + 1)
        assert relrms(back[i], refa[i]) <= TOL, (int(m), relrms(back[i], refa[i]))
