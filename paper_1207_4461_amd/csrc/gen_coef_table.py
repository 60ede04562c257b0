"""Write qbx_coef_table.h: how far two clusters must be apart for the coefficients themselves.

The potential in a disk needs the high coefficients of a far field only as much as J_n(k R)
lets them in (qbx_far_table.h); a caller that keeps the coefficients may read each by itself.
a_n is a sum of terms q H_n(k rho) e^{-i n theta} (S; for D q times (k/2) of the orders n - 1
and n + 1), so its error is measured against the sum of their moduli.  Expansions of order Q
leave out, per unit of q and for all phases at their worst,

  * at the source cluster (radius a, x = k a; the center at distance d, z = k d)
      sum_{|m| > Q} |J_m(x)| |H_{|m| + n}(z)|,
  * at the target cluster (the centers within a of its mean, the source at distance d)
      sum_{|l| > Q} |H_l(z)| |J_{l - n}(x)|,

with J (source) or H (target) replaced by the sum of its neighbours for D.  Entries
[p][i] are the smallest z at which both kinds' sums are below TOL times |H_n(z + x)| (D: the
sum of its neighbours) for n = 0..p and x = 2^(I0 + i / STEPS); 1e300 where no z is.

python gen_coef_table.py > qbx_coef_table.h
"""
import math

import mpmath as mp

TOL = 1e-15
Q = 24
I0, I1, STEPS = -12, 1, 8      # x from 2^-12 to 2
P_MAX = 12
Z_MIN, Z_MAX = 1e-3, 400.0
TAIL = 40                      # terms past Q that are added (they fall by 2 and more each)

mp.mp.dps = 20


def hankels(n, z):
    """|H_0| .. |H_n| at z by the upward recurrence (stable for H)."""
    h = [mp.mpc(mp.besselj(v, z), mp.bessely(v, z)) for v in (0, 1)]
    for v in range(1, n):
        h.append(2 * v / z * h[v] - h[v - 1])
    return [abs(v) for v in h]


def bessels(n, x):
    """|J_0| .. |J_n| at x by the downward recurrence."""
    m = n + 40
    j = [mp.mpf(0)] * (m + 2)
    j[m] = mp.mpf(10) ** -300
    for v in range(m, 0, -1):
        j[v - 1] = 2 * v / x * j[v] - j[v + 1]
    s = mp.besselj(0, x) / j[0] if abs(j[0]) > abs(j[1]) else mp.besselj(1, x) / j[1]
    return [abs(v * s) for v in j[:n + 1]]


def ok(side, n, z, x, J):
    top = Q + TAIL + n + 2
    H, Hc = hankels(top, z), hankels(n + 1, z + x)
    lead = (Hc[n], Hc[abs(n - 1)] + Hc[n + 1])
    near = (lambda A, v: A[v], lambda A, v: A[abs(v - 1)] + A[v + 1])
    for kind in (0, 1):
        if side == 0:
            s = sum(2 * near[kind](J, m) * H[m + n] for m in range(Q + 1, Q + TAIL))
        else:
            s = sum(near[kind](H, l) * (J[l - n] + J[l + n]) for l in range(Q + 1, Q + TAIL))
        if s > TOL * lead[kind]:
            return False
    return True


def zmin(side, n, x):
    J = bessels(Q + TAIL + n + 2, x)
    lo, hi = math.log(Z_MIN), math.log(Z_MAX)
    if ok(side, n, mp.mpf(Z_MIN), x, J):
        return Z_MIN
    if not ok(side, n, mp.mpf(Z_MAX), x, J):
        return None
    while hi - lo > 1e-4:
        mid = 0.5 * (lo + hi)
        if ok(side, n, mp.e ** mid, x, J):
            hi = mid
        else:
            lo = mid
    return math.exp(hi)


def main():
    n = (I1 - I0) * STEPS + 1
    print("// Generated by gen_coef_table.py: the smallest z = k d at which expansions of order %d give"
          % Q)
    print("// the coefficients up to order p (row p) to %g of their terms' moduli." % TOL)
    print("#pragma once")
    print("namespace qbx {")
    print("namespace coeftab {")
    print("constexpr int kI0 = %d, kSteps = %d, kLen = %d, kP = %d;" % (I0, STEPS, n, P_MAX))
    print("}")
    print("}  // namespace qbx")
    for side, name in ((0, "SOURCE"), (1, "TARGET")):
        print("#define QBX_COEF_ZMIN_%s \\" % name)
        best = [0.0] * n
        rows = []
        for p in range(P_MAX + 1):
            for i in range(n):
                if best[i] is not None:
                    v = zmin(side, p, mp.mpf(2) ** (mp.mpf(I0) + mp.mpf(i) / STEPS))
                    best[i] = None if v is None else max(best[i], v)
            rows += ["1e300" if v is None else "%.9g" % v for v in best]
        for i in range(0, len(rows), 8):
            print("  " + ", ".join(rows[i:i + 8]) + (", \\" if i + 8 < len(rows) else ""))


if __name__ == "__main__":
    main()
