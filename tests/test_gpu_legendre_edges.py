"""FP64 Legendre kernels at the edges of their tiles: slot counts around every
change of slots per lane, of workgroups per m and of the polar set, with odd
and even l - m ranges, mmax < lmax and short columns, against the oracle.

Tolerance: 1e-12 relative RMS, the bar of every FP64 result; the recurrence
contributes a few 1e-16 per step at these lmax (below 100 steps)."""
import numpy as np
import pytest

import oracle
import sht_inputs as si

pytestmark = pytest.mark.gpu
TOL = 1e-12


def say(msg):
    print(f"[gpu] {msg}", flush=True)


def relrms(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def rings(nslots, seed, polar):
    """nslots unpaired or mirrored rings; polar: two thirds of them above 45 degrees."""
    rng = np.random.default_rng(seed)
    th = np.sort(rng.uniform(0.01, 0.7 if polar else 1.5, nslots))
    if polar:
        th[::3] = rng.uniform(0.8, 1.55, len(th[::3]))
        th = np.sort(th)
    south = (np.longdouble("3.14159265358979323846264338327950288") - th[: nslots // 2]).astype(np.float64)
    theta = np.concatenate([th, south])
    order = np.argsort(theta)
    n = len(theta)
    nphi = np.full(n, 9)
    return si._pack(theta[order], nphi, rng.uniform(-1, 4, n), rng.uniform(0.1, 1.0, n), f"edge{nslots}")


CASES = [(n, lmax, mmax) for n, lmax, mmax in
         [(1, 9, 9), (63, 40, 40), (64, 41, 30), (65, 37, 37), (128, 38, 38), (129, 6, 6), (255, 33, 20), (256, 34, 34),
          (257, 35, 35), (512, 36, 36), (513, 39, 39), (768, 32, 11), (769, 31, 31), (1024, 30, 30), (1025, 29, 29),
          (1537, 28, 28), (2048, 27, 27), (2049, 26, 26)]]


@pytest.mark.parametrize("nslots,lmax,mmax", CASES)
def test_slot_count_edges(nslots, lmax, mmax):
    import torch
    import paper_1106_0159_amd as sht
    for polar in (False, True):
        g = rings(nslots, 100 + nslots, polar)
        assert sht.ring_slots(g.theta) == nslots
        a = si.uniform_alm(lmax, mmax, nslots)
        s = si.random_map(g, nslots)
        ref, ref_a = oracle.alm2map(lmax, mmax, g, a), oracle.map2alm(lmax, mmax, g, s)
        for nmaps in (1, 3):
            say(f"edges: {nslots} slots polar={polar} lmax={lmax} mmax={mmax} nmaps={nmaps}")
            mp = sht.alm2map(torch.from_numpy(np.stack([a] * nmaps)).cuda(), g, lmax, mmax).cpu().numpy()
            al = sht.map2alm(torch.from_numpy(np.stack([s] * nmaps)).cuda(), g, lmax, mmax).cpu().numpy()
            for k in range(nmaps):
                assert relrms(mp[k], ref) <= TOL, (nslots, polar, k, relrms(mp[k], ref))
                assert relrms(al[k], ref_a) <= TOL, (nslots, polar, k, relrms(al[k], ref_a))


@pytest.mark.parametrize("nslots,tile", [(64, 1), (128, 2), (256, 4), (256, 17), (300, 18), (1100, 20)])
def test_batch_tiles_with_polar_slots(nslots, tile):
    """Batch analysis tiles on grids that are mostly polar (with 256 slots
    every slot of a wave tile is), synthesis bitwise the single call."""
    import torch
    import paper_1106_0159_amd as sht
    lmax = 25
    g = rings(nslots, 7, True)
    if nslots == 256:
        g = si._pack(np.linspace(0.02, 0.75, nslots), np.full(nslots, 9), np.zeros(nslots), np.ones(nslots), "cap")
    a, s = si.uniform_alm(lmax, lmax, 3), si.random_map(g, 4)
    say(f"batch: {nslots} polar slots, tile {tile}")
    b = sht.Batch([("map2alm", lmax, g, torch.from_numpy(s).cuda(), None, tile),
                   ("alm2map", lmax, g, torch.from_numpy(a).cuda(), None)])
    b.run()
    torch.cuda.synchronize()
    got, mp = (o.cpu().numpy() for o in b.outputs)
    b.close()
    ref = oracle.map2alm(lmax, lmax, g, s)
    assert relrms(got, ref) <= TOL, relrms(got, ref)
    assert np.array_equal(mp, sht.alm2map(torch.from_numpy(a).cuda(), g, lmax).cpu().numpy())


@pytest.mark.parametrize("nslots,nmaps", [(65, 3), (255, 4), (256, 5), (257, 6), (512, 9), (513, 4), (769, 5), (1024, 3),
                                          (1025, 4), (1537, 6), (2048, 4), (2049, 3), (2049, 5), (4097, 4)])
def test_many_maps(nslots, nmaps):
    """Analysis of several maps: sets per wave, workgroups per m and maps left
    over, every map a different one."""
    import torch
    import paper_1106_0159_amd as sht
    for polar, lmax, mmax in ((False, 37, 37), (True, 30, 11), (True, 4, 4)):
        g = rings(nslots, 300 + nslots, polar)
        s = np.stack([si.random_map(g, 10 * nslots + k) for k in range(nmaps)])
        say(f"many maps: {nslots} slots polar={polar} lmax={lmax} mmax={mmax} nmaps={nmaps}")
        al = sht.map2alm(torch.from_numpy(s).cuda(), g, lmax, mmax).cpu().numpy()
        for k in range(nmaps):
            ref = oracle.map2alm(lmax, mmax, g, s[k])
            assert relrms(al[k], ref) <= TOL, (nslots, polar, lmax, k, relrms(al[k], ref))


def test_many_maps_infinite_ring():
    """An infinite pixel stays in its map, and out of the columns and degrees
    before its ring's start, as with one map."""
    import torch
    import paper_1106_0159_amd as sht
    g = rings(300, 11, False)
    s = np.stack([si.random_map(g, k) for k in range(4)])
    s[1, 0] = np.inf  # a pixel of the ring nearest the pole
    al = sht.map2alm(torch.from_numpy(s).cuda(), g, 400).cpu().numpy()
    one = sht.map2alm(torch.from_numpy(s[1:2]).cuda(), g, 400).cpu().numpy()
    for k in (0, 2, 3):
        assert relrms(al[k], oracle.map2alm(400, 400, g, s[k])) <= TOL
    assert np.isfinite(one).any() and not np.isfinite(one).all()
    # a set of 64 slots shares its first start: other degrees may be lost only
    # in the orders in which the ring has a term at all
    for m in range(401):
        base = m * (2 * 400 + 1 - m) // 2
        col = slice(base + m, base + 401)
        if np.isfinite(one[0][col]).all():
            assert np.isfinite(al[1][col]).all(), m
