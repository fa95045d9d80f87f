"""Legendre stage in long double (numpy), for rings where the arithmetic of a
double-precision reference is itself in question.  Straight from the
definitions: lambda_mm = (-1)^m mu_m sin^m(theta), lambda_lm = beta_lm (x
lambda_{l-1,m} - lambda_{l-2,m} / beta_{l-1,m}), beta_lm = sqrt((4 l^2 - 1) /
(l^2 - m^2)), cos and sin of the given (double) colatitude in long double."""
import numpy as np

import sht_inputs as si

L = np.longdouble


def legendre_rows(lmax, mmax, theta):
    """Yields (l, lambda) for l = 0..lmax, lambda[r, m] for m = 0..min(l, mmax)."""
    th = np.asarray(theta, dtype=np.float64).astype(L)
    x, s = np.cos(th)[:, None], np.sin(th)
    m2 = np.arange(mmax + 1).astype(L) ** 2
    p1 = p2 = np.zeros((len(th), mmax + 1), dtype=L)
    b1 = np.ones(mmax + 1, dtype=L)
    mm = np.full(len(th), 1 / np.sqrt(4 * np.arccos(L(-1))), dtype=L)
    for l in range(lmax + 1):
        n = min(l, mmax + 1)  # m < n have l > m
        p = np.zeros_like(p1)
        l2 = L(l) * l
        b = np.ones(mmax + 1, dtype=L)
        b[:n] = np.sqrt((4 * l2 - 1) / (l2 - m2[:n]))
        p[:, :n] = b[:n] * (x * p1[:, :n] - p2[:, :n] / b1[:n])
        if l <= mmax:
            if l > 0:
                mm = -mm * s * np.sqrt(L(2 * l + 1) / L(2 * l))
            p[:, l] = mm
        yield l, p[:, : min(l, mmax) + 1]
        p2, p1, b1 = p1, p, b


def alm2delta(lmax, mmax, theta, alm):
    """Delta_m(r) = sum_l a_lm lambda_lm(theta_r), complex long double [nrings, mmax+1]."""
    re, im = (np.zeros((len(theta), mmax + 1), dtype=L) for _ in range(2))
    a = np.asarray(alm)
    for l, p in legendre_rows(lmax, mmax, theta):
        n = p.shape[1]
        c = a[si.alm_index(l, np.arange(n), lmax)]
        re[:, :n] += c.real.astype(L) * p
        im[:, :n] += np.where(np.arange(n) > 0, c.imag, 0.0).astype(L) * p
    return re, im


def delta2alm(lmax, mmax, theta, delta):
    """a_lm = sum_r Delta_m(r) lambda_lm(theta_r), long double (re, im), packed."""
    d = np.asarray(delta)
    dr, di = d.real.astype(L), d.imag.astype(L)
    re, im = (np.zeros(si.nalm(lmax, mmax), dtype=L) for _ in range(2))
    for l, p in legendre_rows(lmax, mmax, theta):
        n = p.shape[1]
        ix = si.alm_index(l, np.arange(n), lmax)
        re[ix] = (dr[:, :n] * p).sum(axis=0)
        im[ix] = np.where(np.arange(n) > 0, (di[:, :n] * p).sum(axis=0), 0.0)
    return re, im
