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
