"""FP64 Legendre stages ring by ring against long double, on rings where the
whole-map error hides them: next to a pole and next to the equator.

Bars, relative RMS of one ring (synthesis) or of the a_lm of one ring
(analysis), all m: next to a pole 1e-12 at lmax 2048.  The recurrence makes
about lmax / 2 steps of two degrees whose roundings (2^-53 each) add up in its
second difference; cos(theta) rounded to a double alone would cost 2^-54 lmax /
sin(theta), 2e-10 on the first ring of HEALPix N_side 1024.  Next to the
equator the roundings of the lmax steps add up as a random walk: with two to
three per step 2^-53 sqrt(3 lmax) = 9e-15 at lmax 2048 and 6e-15 at 1024; the
bar is twice that at the larger, 2e-14."""
import numpy as np
import pytest

import _longdouble as ld
import sht_inputs as si

pytestmark = pytest.mark.gpu
LMAX = 2048


def relrms(got, ref):
    """got: complex128, ref: (re, im) in long double."""
    d = (got.real.astype(np.longdouble) - ref[0]) ** 2 + (got.imag.astype(np.longdouble) - ref[1]) ** 2
    return float(np.sqrt(d.sum() / (ref[0] ** 2 + ref[1] ** 2).sum()))


def check(g, rings, bar, lmax=LMAX):
    """Synthesis and analysis of g on the listed rings."""
    import torch
    import paper_1106_0159_amd as sht
    a = si.powerlaw_alm(lmax, lmax, 9)
    got = sht.alm2delta(torch.from_numpy(a).cuda(), g, lmax).cpu().numpy()
    ref = ld.alm2delta(lmax, lmax, g.theta[rings], a)
    rng = np.random.default_rng(5)
    for i, r in enumerate(rings):
        e = relrms(got[r], (ref[0][i], ref[1][i]))
        print(f"[gpu] {g.name} ring {r} (theta {g.theta[r]:.6f}): synthesis {e:.2e}", flush=True)
        assert e <= bar, (int(r), e)
    for r in rings[:: max(1, len(rings) // 3)]:
        d = np.zeros((g.nrings, lmax + 1), dtype=np.complex128)
        d[r] = rng.standard_normal(lmax + 1) + 1j * rng.standard_normal(lmax + 1)
        back = sht.delta2alm(torch.from_numpy(d).cuda(), g, lmax).cpu().numpy()
        e = relrms(back, ld.delta2alm(lmax, lmax, g.theta[r : r + 1], d[r : r + 1]))
        print(f"[gpu] {g.name} ring {r} (theta {g.theta[r]:.6f}): analysis {e:.2e}", flush=True)
        assert e <= bar, (int(r), e)


def test_rings_next_to_a_pole():
    """The first 400 rings of HEALPix N_side 1024."""
    h = si.healpix(1024)
    n = 400
    g = si._pack(h.theta[:n], np.full(n, 4), h.phi0[:n], np.ones(n), "cap400")
    check(g, np.array([0, 1, 2, 5, 20, 60, 127, 128, 200, 255]), 1e-12)


@pytest.mark.parametrize("nslots", [40, 255])
def test_small_polar_cap(nslots):
    """A cap of few rings: the polar form goes by the colatitude of a ring, not by
    how many rings are near it."""
    h = si.healpix(1024)
    g = si._pack(h.theta[:nslots], np.full(nslots, 4), h.phi0[:nslots], np.ones(nslots), f"cap{nslots}")
    check(g, np.array([0, 1, 2, 5, 20, nslots - 1]), 1e-12)


@pytest.mark.parametrize("lmax", [512, 1024, 2048])
@pytest.mark.parametrize("form", ["healpix", "band", "few"])
def test_rings_next_to_the_equator(lmax, form):
    """The equator itself and rings 1e-4 to 3e-2 rad from it: in the HEALPix grid
    of this lmax, in a band of rings around the equator, and among a few rings."""
    off = np.array([0.0, 1e-4, 3e-4, 1e-3, 3e-3, 1e-2, 3e-2])
    if form == "healpix":
        th = si.healpix(lmax // 2).theta
    elif form == "band":
        th = np.pi / 2 - np.linspace(0.0, 0.05, 701)
    else:
        th = np.linspace(0.1, 1.4, 20)
    th = np.unique(np.concatenate([th, np.pi / 2 - off]))
    g = si._pack(th, np.full(len(th), 4), np.zeros(len(th)), np.ones(len(th)), f"equator-{form}-{lmax}")
    check(g, np.searchsorted(th, np.sort(np.pi / 2 - off)), 2e-14, lmax)
