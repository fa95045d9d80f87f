"""A map's results do not depend on the other maps of its call: FP64 synthesis
and analysis of several maps give every map the bits of its own single call,
at every slot count where the Legendre kernels change their form (one wave per
m, slots per lane, workgroups per m) and at every place within the call.

Tolerance: none, the comparison is bitwise."""
import numpy as np
import pytest

import sht_inputs as si

pytestmark = pytest.mark.gpu


def rings(nslots, seed):
    """nslots rings of the northern hemisphere with some mirror images, few pixels each."""
    rng = np.random.default_rng(seed)
    th = np.sort(rng.uniform(0.01, 1.56, nslots))
    south = (np.longdouble("3.14159265358979323846264338327950288") - th[: nslots // 2]).astype(np.float64)
    theta = np.sort(np.concatenate([th, south]))
    n = len(theta)
    return si._pack(theta, rng.integers(5, 12, n).astype(np.int32), rng.uniform(-1, 4, n), rng.uniform(0.1, 1.0, n),
                    f"independent{nslots}")


@pytest.mark.parametrize("nslots", [64, 65, 128, 129, 192, 193, 256, 257, 512, 513, 640, 641, 770, 1024, 1025, 1400, 2048,
                                    2049, 2600])
def test_maps_of_a_call_are_independent(nslots):
    import torch
    import paper_1106_0159_amd as sht
    lmax, mmax, nmaps = 41, 37, 7
    g = rings(nslots, nslots)
    s = np.stack([si.random_map(g, 10 + k) for k in range(nmaps)])
    s[3] = s[6] = s[0]  # one map at several places of a call
    a = np.stack([si.uniform_alm(lmax, mmax, 20 + k) for k in range(nmaps)])
    a[3] = a[6] = a[0]
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    one_a = [sht.map2alm(dev(s[k]), g, lmax, mmax).cpu().numpy() for k in range(nmaps)]
    one_m = [sht.alm2map(dev(a[k]), g, lmax, mmax).cpu().numpy() for k in range(nmaps)]
    for n in (2, 3, 4, 5, 7):
        print(f"[gpu] independence: {nslots} slots, {n} maps", flush=True)
        back = sht.map2alm(dev(s[:n]), g, lmax, mmax).cpu().numpy()
        many = sht.alm2map(dev(a[:n]), g, lmax, mmax).cpu().numpy()
        for k in range(n):
            assert np.array_equal(back[k], one_a[k]), (nslots, n, k)
            assert np.array_equal(many[k], one_m[k]), (nslots, n, k)


def test_infinite_ring_same_in_every_call():
    """An infinite pixel costs a map the same a_lm whether it is alone or not:
    those of its ring's orders from the ring's own start on."""
    import torch
    import paper_1106_0159_amd as sht
    lmax = 400
    g = rings(300, 11)
    s = np.stack([si.random_map(g, k) for k in range(4)])
    s[1, 0] = np.inf
    print("[gpu] independence: infinite pixel", flush=True)
    al = sht.map2alm(torch.from_numpy(s).cuda(), g, lmax).cpu().numpy()
    one = sht.map2alm(torch.from_numpy(s[1:2]).cuda(), g, lmax).cpu().numpy()[0]
    assert np.isfinite(one).any() and not np.isfinite(one).all()
    assert np.array_equal(np.isfinite(al[1]), np.isfinite(one))
    for k in (0, 2, 3):
        assert np.isfinite(al[k]).all()
