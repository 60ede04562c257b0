"""CPU check of the distances from which panel expansions stand for their pairs.

For random clusters as close as the committed table (csrc/qbx_far_table.h) lets them come, the
translated expansion (sources -> multipole -> local -> target) of order 24
is compared with the Hankel function of the distance: the terms left out are below
1e-17 of the leading one, so in double precision only rounding remains: 2e-14 of |H_0| at the nearest point of the two
disks (some 50 terms of either index, each rounded to 1e-16 of at most that).
"""
import os
import re

import numpy as np
import pytest
import scipy.special as sps

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(HERE, "..", "paper_1207_4461_amd", "csrc", "qbx_far_table.h")


def tables():
    txt = open(HEADER).read()
    i0, steps, n = (int(v) for v in re.search(r"kI0 = (-?\d+), kSteps = (\d+), kLen = (\d+)",
                                              txt).groups())
    out = {}
    for order in (24,):
        body = txt.split("#define QBX_FAR_ZMIN_%d" % order)[1].split("#define")[0]
        vals = [float(v) for v in re.findall(r"[0-9][0-9.e+-]*", body)]
        assert len(vals) == n
        out[order] = vals
    return i0, steps, out


def zmin(order, x):
    i0, steps, tab = tables()
    i = int(np.ceil((np.log2(x) - i0) * steps))
    v = np.inf if i >= len(tab[order]) else tab[order][max(i, 0)]
    return v if v < 1e290 else np.inf


def translated(order, k, src, b_a, b_b, y):
    """H_0(k |y - src|) through the expansions about b_a and b_b."""
    v = src - b_a
    D = b_b - b_a
    t = y - b_b
    l = np.arange(-order, order + 1)
    M = sps.jv(l, k * abs(v)) * np.exp(-1j * l * np.angle(v))
    n = l[None, :] - l[:, None]                      # m - l
    F = sps.hankel1(n, k * abs(D)) * np.exp(1j * n * np.angle(D))
    L = F @ M
    return np.sum(L * sps.jv(l, k * abs(t)) * np.exp(1j * l * np.angle(t)))


@pytest.mark.parametrize("x", (2.0 ** -11, 0.01, 0.1, 0.5, 0.9, 2.0, 3.3))
def test_order_resolves_the_distance(x, order=24):
    rng = np.random.default_rng(int(1000 * x) + order)
    k = 1.0
    rt = x
    rs = x * 0.45
    zt, zs = zmin(order, k * rt), zmin(order, k * rs)
    assert np.isfinite(zt)
    d = max(zs + rt, zt + rs) / k
    for _ in range(20):
        a = np.exp(1j * rng.uniform(0, 2 * np.pi))
        D = d * a
        src = rs * np.exp(1j * rng.uniform(0, 2 * np.pi))
        if rng.uniform() < 0.3:
            src = rs * a                              # towards the target: the worst case
        tgt = D + rt * (np.exp(1j * rng.uniform(0, 2 * np.pi)) if rng.uniform() < 0.7 else -a)
        ref = sps.hankel1(0, k * abs(tgt - src))
        got = translated(order, k, src, 0.0, D, tgt)
        # rounding in the translation is relative to the leading term at the nearest point
        scale = abs(sps.hankel1(0, k * (d - rt - rs)))
        assert abs(got - ref) < 2e-14 * max(scale, abs(ref))


def test_tables_grow_with_the_radius():
    _, _, tab = tables()
    assert all(b >= a for a, b in zip(tab[24], tab[24][1:]))
    assert min(tab[24]) >= 1e-3                       # higher orders of H stay finite


# ---------------------------------------------------------------------------
# the coefficients themselves (csrc/qbx_coef_table.h)
# ---------------------------------------------------------------------------
COEF = os.path.join(HERE, "..", "paper_1207_4461_amd", "csrc", "qbx_coef_table.h")


def coef_tables():
    txt = open(COEF).read()
    i0, steps, n, top = (int(v) for v in re.search(
        r"kI0 = (-?\d+), kSteps = (\d+), kLen = (\d+), kP = (\d+)", txt).groups())
    tab = [np.array([float(v) for v in re.findall(
        r"[0-9][0-9.e+-]*", txt.split("#define QBX_COEF_ZMIN_" + name)[1].split("#define")[0])])
        .reshape(top + 1, n) for name in ("SOURCE", "TARGET")]
    return i0, steps, tab


@pytest.mark.parametrize("p", (0, 1, 5, 12))
@pytest.mark.parametrize("x", (2.0 ** -11, 0.03, 0.4, 0.7))
def test_every_order_of_the_coefficients(p, x, order=24):
    """At the nearest distance that the table allows, each a_n, |n| <= p, of S and of D is right
    to 1e-13 of its term's modulus, the per-order bar of expansion_bars.py for one term."""
    i0, steps, tab = coef_tables()
    rng = np.random.default_rng(int(1e4 * x) + p)
    rs, rt = 0.6 * x, x                                # k = 1
    z = [t[p][max(0, int(np.ceil((np.log2(r) - i0) * steps)))] for t, r in zip(tab, (rs, rt))]
    d = max(z[0] + rt, z[1] + rs)
    assert d < 1e290
    l = np.arange(-order, order + 1)
    n = np.arange(-p - 1, p + 2)
    wave = lambda m, v: sps.jv(m, abs(v)) * np.exp(1j * m * np.angle(v))
    for i in range(20):
        a = np.exp(1j * rng.uniform(0, 2 * np.pi))
        u, v = ((1, 1) if i == 0 else np.exp(2j * np.pi * rng.uniform(size=2)))
        src, tau, D, nu = rs * a * u, -rt * a * v, d * a, np.exp(2j * np.pi * rng.uniform())
        F = sps.hankel1(l[None, :] - l[:, None], d) * np.exp(1j * (l[None, :] - l[:, None]) * np.angle(D))
        g = np.conj(wave(np.arange(-order - 1, order + 2), src))
        M = {"S": g[1:-1], "D": 0.5 * (np.conj(nu) * g[:-2] - nu * g[2:])}
        w = src - (D + tau)
        f = sps.hankel1(n, abs(w)) * np.exp(-1j * n * np.angle(w))
        h = abs(f)
        exact = {"S": f[1:-1], "D": 0.5 * (np.conj(nu) * f[:-2] - nu * f[2:])}
        bound = {"S": h[1:-1], "D": 0.5 * (h[:-2] + h[2:])}
        for kind in "SD":
            L = F @ M[kind]
            got = np.array([np.sum(L * wave(l - m, tau)) for m in n[1:-1]])
            assert (abs(got - exact[kind]) <= 1e-13 * bound[kind]).all()


def test_coefficient_tables_grow():
    for t in coef_tables()[2]:
        assert (np.diff(t, axis=0) >= 0).all()                       # with the order
        ok = np.diff(t, axis=1) >= -1e-3 * t[:, :-1]                 # with the radius
        assert ok.all() and t.min() >= 1e-3
