"""Write qbx_log_table.h: the table of the logarithm in the small-argument Hankel seeds.

For z = 2^e m, 1 <= m < 2, and i the leading 8 bits of m's fraction:
ln(z/2) + gamma = e ln 2 + t_i + ln(1 + r), r = m c_i - 1, with c_i the double nearest to the
reciprocal of interval i's midpoint and t_i = gamma - ln 2 - ln c_i (of the rounded c_i, 40 digits,
rounded once); |r| < 2^-9.

python gen_log_table.py > qbx_log_table.h
"""
import mpmath as mp

mp.mp.dps = 40
N = 256


def main():
    print("// Generated by gen_log_table.py: c_i, t_i with ln(z/2) + gamma = e ln 2 + t_i + ln(m c_i).")
    print("#pragma once")
    print("namespace qbx {\nnamespace logtab {")
    print("constexpr int kN = %d;" % N)
    print("}\n}  // namespace qbx")
    print("#define QBX_LOG_TABLE_VALUES \\")
    rows = []
    for i in range(N):
        c = float(1 / (1 + (mp.mpf(i) + mp.mpf(1) / 2) / N))
        t = mp.euler - mp.log(2) - mp.log(mp.mpf(c))
        rows.append("%.17g, %.17g" % (c, float(t)))
    print(", \\\n".join("  " + ", ".join(rows[i:i + 2]) for i in range(0, N, 2)))


if __name__ == "__main__":
    main()
