"""Rounding of the recursion's stage (eri4_hermite_r), which runs the code of the
integral kernels: no larger than that of the textbook order of the same steps in
doubles, [0]^(m) by repeated products and eq. (md1) level by level, both against
eq. (md1) in extended precision (80 bits, 11 more than a double's).

Bound: the geometric mean over the points of the largest error, relative to the size
that the terms reach (eq. (md1) on absolute values), at most 1.05 times the textbook's:
the mean of 150 such values moves by some 3% with the points drawn.
"""
import numpy as np
import pytest
import torch

from oracle import boys
from paper_2307_03452_amd import eri4

pytestmark = pytest.mark.gpu
LD = np.longdouble


def boys_long(mmax, T):
    """F_m(T) in extended precision: the (all positive) series below 60, upward
    recursion from it above, where exp(-T) is below the last bit."""
    T = LD(T)
    if T < 60:
        term = LD(1) / (2 * mmax + 1)
        s = term
        for k in range(1, 600):
            term *= 2 * T / (2 * mmax + 2 * k + 1)
            s += term
            if term < s * LD(1e-22):
                break
        F = np.zeros(mmax + 1, LD)
        ex = np.exp(-T)
        F[mmax] = ex * s
        for m in range(mmax - 1, -1, -1):
            F[m] = (2 * T * F[m + 1] + ex) / (2 * m + 1)
        return F
    F = np.zeros(mmax + 1, LD)
    F[0] = np.sqrt(LD("3.14159265358979323846264338327950288") / T) / 2
    for m in range(mmax):
        F[m + 1] = (2 * m + 1) * F[m] / (2 * T)
    return F


def levels(base, pq, L, dtype):
    """[r]^(0) by eq. (md1) from [0]^(m): R[t, u, v]."""
    R = np.zeros((L + 1,) * 3, dtype)
    R[0, 0, 0] = base[L]
    for m in range(L - 1, -1, -1):
        N = np.zeros_like(R)
        for n in range(1, L - m + 1):
            for t in range(n + 1):
                for u in range(n - t + 1):
                    a = [t, u, n - t - u]
                    x = 2 if a[2] > 0 else (1 if a[1] > 0 else 0)
                    r = a[x]
                    a[x] -= 1
                    v = pq[x] * R[tuple(a)]
                    if r > 1:
                        a[x] -= 1
                        v = v + (r - 1) * R[tuple(a)]
                    N[t, u, n - t - u] = v
        N[0, 0, 0] = base[m]
        R = N
    return R


@pytest.mark.parametrize("L,n", [(8, 150), (12, 150), (16, 60)])
def test_no_more_rounding_than_level_by_level(L, n):
    r = np.random.default_rng(L)
    z = np.exp(r.uniform(np.log(0.05), np.log(200.0), (4, n)))
    c = r.uniform(0.0, 8.0, (4, n, 3))
    zp, zq = z[0] + z[1], z[2] + z[3]
    P = (z[0][:, None] * c[0] + z[1][:, None] * c[1]) / zp[:, None]
    Q = (z[2][:, None] * c[2] + z[3][:, None] * c[3]) / zq[:, None]
    up = lambda x: torch.tensor(np.ascontiguousarray(x)).cuda()  # noqa: E731
    got = eri4.hermite_r(L, up(zp), up(zq), up(P), up(Q)).cpu().numpy()
    mine, textbook = [], []
    for i in range(n):
        pq = P[i] - Q[i]
        rho, r2 = LD(zp[i]) * LD(zq[i]) / (LD(zp[i]) + LD(zq[i])), sum(LD(x) * LD(x) for x in pq)
        pref = 2 * LD("17.4934183276248628462628216798715530") / (LD(zp[i]) * LD(zq[i]) * np.sqrt(LD(zp[i]) + LD(zq[i])))
        base = np.array([(-2 * rho) ** m for m in range(L + 1)]) * pref * boys_long(L, rho * r2)
        ref = levels(base, [LD(x) for x in pq], L, LD)
        mag = levels(np.abs(base), [abs(LD(x)) for x in pq], L, LD)
        mag[mag < 1e-290] = np.inf
        rd = zp[i] * zq[i] / (zp[i] + zq[i])
        F = boys(L, float(rd * (pq[0] * pq[0] + pq[1] * pq[1] + pq[2] * pq[2])))
        pd, bd, pw = 2.0 * np.pi ** 2.5 / (zp[i] * zq[i] * np.sqrt(zp[i] + zq[i])), np.zeros(L + 1), 1.0
        for m in range(L + 1):
            bd[m] = pw * pd * F[m]
            pw *= -2.0 * rd
        mine.append(float(np.max(np.abs(got[i] - ref) / mag)))
        textbook.append(float(np.max(np.abs(levels(bd, pq, L, np.float64) - ref) / mag)))
    a, b = np.exp(np.mean(np.log(mine))), np.exp(np.mean(np.log(textbook)))
    assert a <= 1.05 * b, (a, b)


def test_high_orders_of_distant_pairs_keep_their_digits():
    """[0]^(m) above the Boys table is (-2 / r^2)^m times a constant: with P - Q along
    z, R[2i, 2j, 0] = (2i-1)!! (2j-1)!! [0]^(i+j).  Bound: m + 6 roundings of half a unit
    (the square r^2 enters m times, the quotient another m, both of random sign)."""
    L, n = 28, 400
    r = np.random.default_rng(3)
    zp, zq = r.uniform(5.0, 300.0, n), r.uniform(5.0, 300.0, n)
    d = r.uniform(8.0, 30.0, n)
    P, Q = np.zeros((n, 3)), np.zeros((n, 3))
    P[:, 2] = d
    up = lambda x: torch.tensor(np.ascontiguousarray(x)).cuda()  # noqa: E731
    got = eri4.hermite_r(L, up(zp), up(zq), up(P), up(Q)).cpu().numpy()
    odd = lambda k: np.prod(np.arange(1, 2 * k, 2, dtype=LD)) if k else LD(1)  # noqa: E731
    for m in (4, 8, 14):
        err = []
        for i in range(n):
            rho, r2 = LD(zp[i]) * LD(zq[i]) / (LD(zp[i]) + LD(zq[i])), LD(d[i]) ** 2
            pref = 2 * LD("17.4934183276248628462628216798715530") / (LD(zp[i]) * LD(zq[i]) * np.sqrt(LD(zp[i]) + LD(zq[i])))
            ref = (-2 * rho) ** m * pref * boys_long(m, rho * r2)[m] * odd(m)
            err.append(float(abs(got[i, 2 * m, 0, 0] - ref) / abs(ref)))
        # rms: sqrt(2) m errors of 0.29 units in the last place (2^-52 at most) and the rest
        rms = np.sqrt(np.mean(np.square(err)))
        assert rms <= 0.29 * 2.0 ** -52 * np.sqrt(2.0 * m * m + 6.0), (m, rms / 2.0 ** -52)
