"""Write qbx_far_table.h: how far two clusters must be apart for expansions of a given order.

For a cluster of radius a (x = k a) the terms of its multipole (or local) expansion at a
distance d (z = k d) are bounded by |J_m(x)| |H_m(z)| <= (x/2)^m / m! |H_m(z)|, and
|H_m(z)| / |H_0(z)| falls with z.  ZMIN(order)[i] is the smallest z at which the term of
order n = order - 1 is below TOL |H_0(z)| for x = 2^(I0 + i / STEPS); the expansions keep
the orders |m| <= order, so that two orders beyond n (and with them the first and second
derivatives of the sums, each a factor of about n d / a) are still below it.
A value that no z up to Z_MAX meets is written as infinity.

python gen_far_table.py > qbx_far_table.h
"""
import math

import mpmath as mp

TOL = 1e-17
I0, I1, STEPS = -12, 5, 8      # x from 2^-12 to 2^5
ORDERS = (24,)
Z_MIN, Z_MAX = 1e-3, 2000.0    # below Z_MIN the high orders of H would overflow

mp.mp.dps = 30


def ok(n, x, z):
    h = mp.sqrt(mp.besselj(n, z) ** 2 + mp.bessely(n, z) ** 2)
    h0 = mp.sqrt(mp.besselj(0, z) ** 2 + mp.bessely(0, z) ** 2)
    return (x / 2) ** n / mp.factorial(n) * h <= TOL * h0


def zmin(n, x):
    lo, hi = math.log(Z_MIN), math.log(Z_MAX)
    x = mp.mpf(x)
    if ok(n, x, mp.e ** lo):
        return Z_MIN
    if not ok(n, x, mp.e ** hi):
        return None
    for _ in range(30):
        mid = 0.5 * (lo + hi)
        if ok(n, x, mp.e ** mid):
            hi = mid
        else:
            lo = mid
    return math.exp(hi) * (1.0 + 1e-6)


def main():
    n = (I1 - I0) * STEPS + 1
    print("// Generated by gen_far_table.py: the smallest z = k d at which a cluster of radius a,")
    print("// x = k a, is resolved by expansions of the order named (term bound %g)." % TOL)
    print("#pragma once")
    print("namespace qbx {")
    print("namespace fartab {")
    print("constexpr int kI0 = %d, kSteps = %d, kLen = %d;" % (I0, STEPS, n))
    print("}")
    print("}  // namespace qbx")
    for o in ORDERS:
        vals = [zmin(o - 1, 2.0 ** (I0 + i / STEPS)) for i in range(n)]
        print("#define QBX_FAR_ZMIN_%d \\" % o)
        txt = ["1e300" if v is None else "%.9g" % v for v in vals]
        for i in range(0, n, 8):
            print("  " + ", ".join(txt[i:i + 8]) + (", \\" if i + 8 < n else ""))


if __name__ == "__main__":
    main()
