"""Write qbx_gl_table.h: the Gauss-Legendre rules of 16, 32, .., 128 points.

Nodes are the roots of P_n by Newton's method at 40 digits, weights
2 / ((1 - x^2) P_n'(x)^2) (DLMF 3.5.30 with table 3.5.1), each rounded to double once.  The rules
are symmetric: the header holds the n/2 positive nodes (ascending) and their weights, for
n = 16, 32, .. in turn; rule n starts at (n/16 - 1) (n/16) / 2 * 8.

python gen_gl_table.py > qbx_gl_table.h
"""
import mpmath as mp

mp.mp.dps = 40


def legendre(n, x):
    p0, p1 = mp.mpf(1), x
    for j in range(1, n):
        p0, p1 = p1, ((2 * j + 1) * x * p1 - j * p0) / (j + 1)
    return p1, n * (x * p1 - p0) / (x * x - 1)


def rule(n):
    out = []
    for i in range(n // 2):
        x = mp.cos(mp.pi * (i + mp.mpf(3) / 4) / (n + mp.mpf(1) / 2))
        for _ in range(12):
            p, d = legendre(n, x)
            x -= p / d
        _, d = legendre(n, x)
        out.append((x, 2 / ((1 - x * x) * d * d)))
    return out[::-1]


def main():
    xs, ws = [], []
    for n in range(16, 129, 16):
        for x, w in rule(n):
            xs.append(x)
            ws.append(w)
    print("// Generated by gen_gl_table.py: positive Gauss-Legendre nodes and weights, 16 .. 128 points.")
    print("#pragma once")
    print("namespace qbx {")
    print("namespace gltab {")
    print("constexpr int kLen = %d;" % len(xs))
    print("}")
    print("}  // namespace qbx")
    for name, v in (("QBX_GL_NODES", xs), ("QBX_GL_WEIGHTS", ws)):
        print("#define %s \\" % name)
        t = ["%.17g" % float(a) for a in v]
        for i in range(0, len(t), 4):
            print("  " + ", ".join(t[i:i + 4]) + (", \\" if i + 4 < len(t) else ""))


if __name__ == "__main__":
    main()
