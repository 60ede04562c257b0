// Panel expansions: the far sums of the pair kernels (derivation in qbx_far.h).
#include "qbx_far.h"
#include "qbx_coef_table.h"
#include "qbx_far_table.h"
#include "qbx_special.h"

namespace qbx {

static __constant__ double g_zmin[fartab::kLen] = {QBX_FAR_ZMIN_24};
static __constant__ double g_coef_zmin[2][coeftab::kP + 1][coeftab::kLen] = {
    {QBX_COEF_ZMIN_SOURCE}, {QBX_COEF_ZMIN_TARGET}};
static_assert(kFarQ == 24, "the tables are for this order");
static_assert(kFarMaxCoefOrder == coeftab::kP, "a row for every order");

// the entry of k radius x (rounded up), or infinity past the table
__device__ __forceinline__ double far_entry(const double* tab, int i0, int steps, int len,
                                            double x) {
  const double s = ceil((log2(fmax(x, 1e-30)) - i0) * steps);
  if (!(s < (double)len)) return 1e300;
  return tab[s > 0.0 ? (int)s : 0];
}
// smallest k d that resolves a cluster of k radius x for the sums at the targets, and as
// sources (side 0) or centers (side 1) for the coefficients up to order p (none past the table)
__device__ __forceinline__ double far_zmin(double x) {
  return far_entry(g_zmin, fartab::kI0, fartab::kSteps, fartab::kLen, x);
}
__device__ __forceinline__ double far_coef_zmin(int side, int p, double x) {
  if (p > coeftab::kP) return 1e300;
  return far_entry(g_coef_zmin[side][p], coeftab::kI0, coeftab::kSteps, coeftab::kLen, x);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  return v;
}
__device__ __forceinline__ double wave_add(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Cluster records, one wave per panel and per group.
__global__ __launch_bounds__(64) void k_far_recs(FarBlocks B, const double* __restrict__ ro,
                                                 const double* __restrict__ nodes,
                                                 double* __restrict__ wo) {
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int lane = threadIdx.x;
  const bool group = b >= it.P;
  const int c = group ? b - it.P : b;
  const int m0 = group ? c * it.g : c;
  const int m1 = group ? min(m0 + it.g, it.P) : c + 1;
  const double* X = nodes + it.node_off;
  double sx = 0.0, sy = 0.0;
  for (int a = m0 * kQ + lane; a < m1 * kQ; a += kWave) {
    sx += X[2 * a];
    sy += X[2 * a + 1];
  }
  const double inv = 1.0 / ((m1 - m0) * kQ);
  const double bx = wave_add(sx) * inv, by = wave_add(sy) * inv;
  double rs = 0.0, rt = 0.0, rb = 0.0, gr = 0.0;
  const double4* geo = reinterpret_cast<const double4*>(ro + it.fgeo);
  for (int j = m0 * it.fqs + lane; j < m1 * it.fqs; j += kWave) {
    const double dx = geo[j].x - bx, dy = geo[j].y - by;
    rs = fmax(rs, sqrt(dx * dx + dy * dy));
  }
  if (it.pt) {
    rt = rs;   // the targets are the far sources' points
  } else {
    const CenterRec* ctr = reinterpret_cast<const CenterRec*>(ro + it.ctr);
    for (int si = 0; si < it.n_sides; ++si)
      for (int t = m0 * kQ + lane; t < m1 * kQ; t += kWave) {
        const CenterRec& C = ctr[(size_t)si * it.T + t];
        const double dx = C.cx - bx, dy = C.cy - by;
        rt = fmax(rt, sqrt(dx * dx + dy * dy) + (it.coef < 0 ? C.R : 0.0));
      }
  }
  if (group && it.pt) {
    const double4* bnd = reinterpret_cast<const double4*>(ro + it.bnd);
    if (m0 + lane < m1) {
      const double4 q = bnd[m0 + lane];
      const double dx = q.x - bx, dy = q.y - by;
      rb = sqrt(dx * dx + dy * dy);
      gr = sqrt(it.g2) * q.w;
    }
  }
  const double up = 1.0 + 1e-12;   // over the rounding of the distances
  rs = wave_max(rs) * up;
  rt = wave_max(rt) * up;
  rb = wave_max(rb) * up;
  gr = wave_max(gr) * up;
  if (lane == 0) {
    FarRec r;
    r.bx = bx;
    r.by = by;
    r.rs = rs;
    r.rt = rt;
    r.ds = (it.coef < 0 ? far_zmin(it.k * rs) : far_coef_zmin(0, it.coef, it.k * rs)) / it.k;
    r.dt = (it.coef < 0 ? far_zmin(it.k * rt) : far_coef_zmin(1, it.coef, it.k * rt)) / it.k;
    r.rb = rb;
    r.gr = gr;
    reinterpret_cast<FarRec*>(wo + (group ? it.rec1 : it.rec0))[c] = r;
  }
}

// J_l(x) = S_l (x/2)^l / l!.  The recurrence of J becomes
// S_{l-1} = S_l - (x^2/4) / (l (l + 1)) S_{l+1}, which neither over- nor underflows;
// started well above the orders wanted it gives S up to a factor, fixed by
// 1 = J_0 + 2 (J_2 + J_4 + ...).  x is at most 2^1.75 = 3.4 for a cluster that
// any distance resolves at order kFarQ (the table ends there: past it the first term left out is
// above 1e-17 at every distance); others are not expanded (far_none).
__device__ __forceinline__ int far_start(double x) {
  x = fmin(x, 64.0);   // bounded work for any argument
  return (int)(x + 16.0 + 4.0 * sqrt(x));
}
__device__ __forceinline__ bool far_none(const FarRec& r) {
  return !(r.ds < 1e290 && r.dt < 1e290);
}

// J[0..L] in registers, L a constant
template <int L>
__device__ __forceinline__ void far_bessel(double x, double (&J)[L + 1]) {
  const double q = 0.25 * x * x;
  const int n0 = max(L + 6, far_start(x));
  double sp = 1.0, sc = 1.0;   // S_{l+1}, S_l at l = n0
  double tail = 0.0;           // sum of J_l / ((x/2)^L / L!) over even l > L, from the top
  for (int l = n0; l > L; --l) {
    if ((l & 1) == 0) tail += sc;
    const double sm = fma(-q * (1.0 / ((double)l * (l + 1))), sp, sc);
    sp = sc;
    sc = sm;
    // the sum below carries (x/2)^l / l! relative to the next lower order
    tail *= 0.5 * x / l;
  }
  // here sc = S_L, sp = S_{L+1}, tail = sum_{even l > L} S_l (x/2)^{l-L} L! / l!
#pragma unroll
  for (int l = L; l >= 0; --l) {
    J[l] = sc;
    if (l > 0) {
      const double sm = fma(-q * (1.0 / ((double)l * (l + 1))), sp, sc);
      sp = sc;
      sc = sm;
    }
  }
  double pw = 1.0, norm = 0.0;
#pragma unroll
  for (int l = 0; l <= L; ++l) {
    if (l > 0) pw *= x * (0.5 / l);
    J[l] *= pw;
    if (l == 0) norm += J[0];
    else if ((l & 1) == 0) norm = fma(2.0, J[l], norm);
  }
  norm = fma(2.0 * pw, tail, norm);
  const double s = 1.0 / norm;
#pragma unroll
  for (int l = 0; l <= L; ++l) J[l] *= s;
}

// J_l into out[l * stride], l <= L (run-time L)
__device__ __forceinline__ void far_bessel_mem(double x, int L, double* __restrict__ out,
                                               int stride) {
  const double q = 0.25 * x * x;
  const int n0 = max(L + 6, far_start(x));
  double sp = 1.0, sc = 1.0, tail = 0.0;
  for (int l = n0; l > 0; --l) {
    if (l <= L) out[l * stride] = sc;
    else if ((l & 1) == 0) tail += sc;
    const double sm = fma(-q * (1.0 / ((double)l * (l + 1))), sp, sc);
    sp = sc;
    sc = sm;
    if (l > L) tail *= 0.5 * x / l;
  }
  double pw = 1.0, norm = sc;
  out[0] = sc;
  for (int l = 1; l <= L; ++l) {
    pw *= x * (0.5 / l);
    const double v = out[l * stride] * pw;
    out[l * stride] = v;
    if ((l & 1) == 0) norm = fma(2.0, v, norm);
  }
  norm = fma(2.0 * pw, tail, norm);
  const double s = 1.0 / norm;
  for (int l = 0; l <= L; ++l) out[l * stride] *= s;
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }

// Sources to multipoles: one wave per panel and per group, one lane per source.  Bound
// by the reduction of the 2 kFarQ + 1 terms over the lanes, which goes through LDS
// (written per lane, then added by one lane per order).
// rows[v][0][c][m] = M_m, rows[v][1][c][m] = (-1)^m M_{-m} (the reflected half of k_far_m2l)
__global__ __launch_bounds__(64) void k_far_p2m(FarBlocks B, const double* __restrict__ ro,
                                                double* __restrict__ wo) {
  __shared__ double2 val[kFarW][kWave + 1];
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  if (far_off(it)) return;
  const int lane = threadIdx.x;
  const bool group = b >= it.P;
  const int c = group ? b - it.P : b;
  const int C = group ? it.C1 : it.P;
  const FarRec rec = reinterpret_cast<const FarRec*>(ro + (group ? it.rec1 : it.rec0))[c];
  const int j0 = (group ? c * it.g : c) * it.fqs;
  const int j1 = group ? min(j0 + it.g * it.fqs, it.P * it.fqs) : j0 + it.fqs;
  const int Nf = it.P * it.fqs;
  const double4* geo = reinterpret_cast<const double4*>(ro + it.fgeo);
  const double2* dens = reinterpret_cast<const double2*>(ro + it.fdens);
  double2* rows = reinterpret_cast<double2*>(wo + (group ? it.rows1 : it.rows0));
  const bool none = far_none(rec);
  for (int kk = 0; kk < it.vf; ++kk) {
    const bool dbl = it.kind == 2 || kk == 1;
    double2 acc = make_double2(0.0, 0.0);   // lane m: M_{m - kFarQ}
    for (int s0 = j0; s0 < j1 && !none; s0 += kWave) {
      const int j = s0 + lane;
      const bool on = j < j1;
      const int jj = on ? j : j1 - 1;
      const double4 g = geo[jj];
      double2 q = dens[(size_t)kk * Nf + jj];
      if (!on) q = make_double2(0.0, 0.0);
      const double vx = g.x - rec.bx, vy = g.y - rec.by;
      const double r2 = fma(vx, vx, vy * vy);
      const double r = sqrt(r2);
      const double2 e = r > 0.0 ? make_double2(vx / r, -vy / r) : make_double2(1.0, 0.0);
      double J[kFarQ + 2];
      far_bessel<kFarQ + 1>(it.k * r, J);
      __syncthreads();
      if (!dbl) {
        double2 w = q;   // q e^{-i m alpha}; the reflected one runs alongside
        double2 u = q;
#pragma unroll
        for (int m = 0; m <= kFarQ; ++m) {
          val[kFarQ + m][lane] = make_double2(w.x * J[m], w.y * J[m]);
          const double jn = (m & 1) ? -J[m] : J[m];
          if (m > 0) val[kFarQ - m][lane] = make_double2(u.x * jn, u.y * jn);
          w = cmul(w, e);
          u = cmul(u, conj2(e));
        }
      } else {
        // d/dnu g_m = (k/2)(conj(nu) g_{m-1} - nu g_{m+1}), g_m = J_m e^{-i m alpha}
        const double hk = 0.5 * it.k;
        const double2 nu = make_double2(hk * g.z, hk * g.w);
        const double2 qa = cmul(q, conj2(nu)), qb = cmul(q, nu);
        // per order m >= 0: e^{-i m alpha}; at order -m its conjugate with (-1)^m
        double2 em = make_double2(e.x, -e.y);   // e^{-i(m-1) alpha} at m = 0
#pragma unroll
        for (int m = 0; m <= kFarQ; ++m) {
          const double2 ec = cmul(em, e), ep = cmul(ec, e);   // m, m + 1
          // J_{m-1} for m = 0 is J_{-1} = -J_1
          const double jm = m == 0 ? -J[1] : J[m > 0 ? m - 1 : 0];
          const double jp = J[m + 1];
          const double2 gm = make_double2(jm * em.x, jm * em.y);
          const double2 gp = make_double2(jp * ep.x, jp * ep.y);
          const double2 a = cmul(qa, gm), bq = cmul(qb, gp);
          val[kFarQ + m][lane] = make_double2(a.x - bq.x, a.y - bq.y);
          if (m > 0) {
            // g_{-m-1} = (-1)^{m+1} conj(g_{m+1}), g_{-m+1} = (-1)^{m-1} conj(g_{m-1})
            const double s = (m & 1) ? 1.0 : -1.0;
            const double2 a2 = cmul(qa, make_double2(s * gp.x, -s * gp.y));
            const double2 b2 = cmul(qb, make_double2(s * gm.x, -s * gm.y));
            val[kFarQ - m][lane] = make_double2(a2.x - b2.x, a2.y - b2.y);
          }
          em = ec;
        }
      }
      __syncthreads();
      if (lane < kFarW) {
        double ar = 0.0, ai = 0.0;
        for (int i = 0; i < kWave; ++i) {
          const double2 v = val[lane][i];
          ar += v.x;
          ai += v.y;
        }
        acc.x += ar;
        acc.y += ai;
      }
    }
    double2* r0 = rows + ((size_t)(kk * 2 + 0) * C + c) * kFarW + kFarQ;
    double2* r1 = rows + ((size_t)(kk * 2 + 1) * C + c) * kFarW + kFarQ;
    if (lane < kFarW) {
      const int m = lane - kFarQ;
      const double s = (m & 1) ? -1.0 : 1.0;
      r0[m] = acc;
      r1[-m] = make_double2(s * acc.x, s * acc.y);
    }
  }
}

// The translation's inner work.  Per pair of clusters and order n of F, L_l takes M_{l+n} F_n
// and M_{l-n} F_{-n}, four FMAs a term with M in scalar registers.  The row (49 complex
// values) does not fit those, so it streams through them in pieces of at most kPiece
// values: the next piece is requested before the current one's FMAs are issued, and its
// latency hides behind them (scalar loads return in any order, so a wait is for all of
// them: the request has to come after the current piece has arrived).  Every order is
// unrolled (45 KB of code); eight rolled blocks of six orders with rows padded to the
// widest (7 KB) were measured 10 to 60% slower at 256 to 4096 panels.
constexpr int kPiece = 8;
struct FarPiece {
  double2 m[kPiece];
};
// order N: F_N serves l < pos, F_{-N} serves l >= neg0
template <int N>
struct FarOrder {
  static constexpr int pos = N <= kFarQ ? kFarQ - N + 1 : 0;
  static constexpr int neg0 = N > kFarQ ? N - kFarQ : 0;
  static constexpr int neg = N == 0 ? 0 : kFarQ + 1 - neg0;
  static constexpr int pp = (pos + kPiece - 1) / kPiece, np = (neg + kPiece - 1) / kPiece;
  static constexpr int pieces = pp + np;
};
// piece PC of order N: M_{m0} .. M_{m0 + len - 1} for l0 ..
template <int N, int PC>
struct FarAt {
  using O = FarOrder<N>;
  static constexpr bool is_pos = PC < O::pp;
  static constexpr int k = is_pos ? PC : PC - O::pp;
  static constexpr int l0 = (is_pos ? 0 : O::neg0) + k * kPiece;
  static constexpr int left = (is_pos ? O::pos : O::neg) - k * kPiece;
  static constexpr int len = left < kPiece ? left : kPiece;
  static constexpr int m0 = is_pos ? l0 + N : l0 - N;
};

// state of one pair's translation: H_{n-1}, H_n, 2n/z, e^{i n phi}
struct FarRun {
  double hm_r, hm_i, hc_r, hc_i, tl, tz;
  double2 E, e;
};

template <int N, int PC>
__device__ __forceinline__ void far_steps(FarRun& f, double fr, double fi, double gr, double gi,
                                          FarPiece cur, const double2* __restrict__ row,
                                          double (&Lr)[kFarQ + 1], double (&Li)[kFarQ + 1]) {
  using A = FarAt<N, PC>;
  constexpr bool last_piece = PC + 1 == FarOrder<N>::pieces;
  constexpr bool last = last_piece && N == 2 * kFarQ;
  constexpr int N2 = last_piece ? N + 1 : N, P2 = last_piece ? 0 : PC + 1;
#pragma unroll
  for (int i = 0; i < A::len; ++i) asm volatile("" : "+s"(cur.m[i].x), "+s"(cur.m[i].y));
  FarPiece nxt;
  if constexpr (!last) {
    using B = FarAt<N2, P2>;
    const double2* __restrict__ r = row + opaque_zero();
#pragma unroll
    for (int i = 0; i < B::len; ++i) nxt.m[i] = r[B::m0 + i];
  }
  __builtin_amdgcn_sched_barrier(0);
  const double Fr = A::is_pos ? fr : gr, Fi = A::is_pos ? fi : gi;
#pragma unroll
  for (int i = 0; i < A::len; ++i) {
    const double2 M = cur.m[i];
    Lr[A::l0 + i] = fma(M.x, Fr, fma(-M.y, Fi, Lr[A::l0 + i]));
    Li[A::l0 + i] = fma(M.x, Fi, fma(M.y, Fr, Li[A::l0 + i]));
  }
  if constexpr (!last) {
    if constexpr (last_piece) {   // F_{n+1}, F_{-n-1}
      const double rr = f.hc_r * f.E.x, ii = f.hc_i * f.E.y, ri = f.hc_r * f.E.y,
                   ir = f.hc_i * f.E.x;
      constexpr double s = (N2 & 1) ? -1.0 : 1.0;
      fr = rr - ii;
      fi = ri + ir;
      gr = s * (rr + ii);
      gi = s * (ir - ri);
      const double hn_r = fma(f.tl, f.hc_r, -f.hm_r), hn_i = fma(f.tl, f.hc_i, -f.hm_i);
      f.hm_r = f.hc_r;
      f.hm_i = f.hc_i;
      f.hc_r = hn_r;
      f.hc_i = hn_i;
      f.tl += f.tz;
      const double er = fma(f.E.x, f.e.x, -f.E.y * f.e.y), ei = fma(f.E.x, f.e.y, f.E.y * f.e.x);
      f.E.x = er;
      f.E.y = ei;
      // one order in flight: without it the compiler runs the recurrences ahead
      asm volatile("" : "+v"(f.hm_r), "+v"(f.hm_i), "+v"(f.hc_r), "+v"(f.hc_i), "+v"(f.E.x),
                   "+v"(f.E.y));
    }
    __builtin_amdgcn_sched_barrier(0);
    far_steps<N2, P2>(f, fr, fi, gr, gi, nxt, row, Lr, Li);
  }
}

// L_l += sum_m M_m F_{m-l}, l = 0..kFarQ, for one pair of clusters a lane; row[m] = M_m,
// wave-uniform
__device__ __forceinline__ void far_translate(double z, double iz, double2 e,
                                              const double2* __restrict__ row,
                                              const double* __restrict__ cf,
                                              double (&Lr)[kFarQ + 1], double (&Li)[kFarQ + 1]) {
  const H01 h = hankel01(z, iz, cf);
  FarRun f{h.h0r, h.h0i, h.h1r, h.h1i, 2.0 * iz, 2.0 * iz, e, e};
  FarPiece first;
#pragma unroll
  for (int i = 0; i < FarAt<0, 0>::len; ++i) first.m[i] = row[i];
  far_steps<0, 0>(f, h.h0r, h.h0i, 0.0, 0.0, first, row, Lr, Li);
}

// Translations: lanes are 64 consecutive target clusters, the source cluster is
// wave-uniform.  One wave takes the orders l >= 0 of one vector; the orders l < 0 are
// those of the reflected problem, (-1)^l L_{-l} = sum_m (-1)^m M_{-m} F_{m-l}(reflected D),
// so the second half runs the same code on the second set of rows with the angle
// negated (half the accumulators in registers, twice the waves).  The four waves of a
// block take every fourth source of the block's share and are added in wave order.
template <bool GROUP>
__global__ __launch_bounds__(256, 3) void k_far_m2l(FarBlocks B, const double* __restrict__ ro,
                                                    double* __restrict__ wo) {
  __shared__ double2 red[kFarQ + 1][kWave];
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  if (far_off(it)) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int C = GROUP ? it.C1 : it.P;
  const int ns = GROUP ? it.n1 : it.n0;
  // block order: source share fastest, then half, vector, target block
  const int sp = b % ns;
  const int half = (b / ns) & 1;
  const int v = (b / (2 * ns)) % it.V;
  const int tb = b / (2 * ns * it.V);
  const FarRec* __restrict__ rec =
      reinterpret_cast<const FarRec*>(ro + (GROUP ? it.rec1 : it.rec0));
  const FarRec* __restrict__ grec = reinterpret_cast<const FarRec*>(ro + it.rec1);
  const double2* __restrict__ rows =
      reinterpret_cast<const double2*>(ro + (GROUP ? it.rows1 : it.rows0)) +
      (size_t)(v * 2 + half) * C * kFarW + kFarQ;
  const bool inner = !GROUP && it.C1 > 0;
  const bool gam = !GROUP && it.pt != 0;
  const int g = it.g;
  double Lr[kFarQ + 1], Li[kFarQ + 1];
#pragma unroll
  for (int l = 0; l <= kFarQ; ++l) Lr[l] = Li[l] = 0.0;
  // One source cluster for the lanes whose pair with it is taken at this level.  The
  // lane's own record is read again each time: it would take registers from the
  // accumulators for the whole loop.
  auto source = [&](int A) {
    const int z0 = opaque_zero();
    const int t = tb * kWave + lane + z0;
    const int tt = t < C ? t : C - 1;
    const FarRec me = rec[tt], o = rec[A];
    bool on = t < C && far_adm(me, o);
    if (inner && on) on = !far_adm(grec[tt / g], grec[A / g]);
    if (gam && on) {
      const double4* bnd = reinterpret_cast<const double4*>(ro + it.bnd);
      on = !panels_near(bnd[tt], bnd[A], it.g2);
    }
    if (!__any(on)) return;
    if (on) {
      const double dx = me.bx - o.bx, dy = me.by - o.by;
      const double d2 = fma(dx, dx, dy * dy);
      const double ir = rsqrt_refined(d2);
      const double k = it.k;
      const double2 e = make_double2(dx * ir, half ? -dy * ir : dy * ir);
      far_translate(k * (d2 * ir), ir / k, e, rows + (size_t)A * kFarW + z0,
                           g_seed_table + z0, Lr, Li);
    }
  };
  const int share = sp * 4 + wave, shares = 4 * ns;
  // Panels whose pairs are mostly taken group by group: a ballot finds the groups that
  // some group of this block's targets does not take (64 at a time), and their panels
  // are dealt out to the waves in turn.  Otherwise every source is a candidate.
  const int end = inner ? it.C1 : C;
  int turn = 0;
#pragma unroll 1
  for (int c0 = inner ? 0 : share; c0 < end; c0 += inner ? kWave : shares) {
    unsigned long long mask = 1;
    if (inner) {
      bool need = false;
      if (c0 + lane < end) {
        const FarRec q = grec[c0 + lane];
        const int t1 = min(tb * kWave + kWave - 1, C - 1) / g;
#pragma unroll 1
        for (int tg = tb * kWave / g; tg <= t1; ++tg) need = need || !far_adm(grec[tg], q);
      }
      mask = __ballot(need);
    }
#pragma unroll 1
    while (mask) {
      const int c = c0 + __builtin_ctzll(mask);
      mask &= mask - 1;
      int A = inner ? c * g : c;
      const int a1 = inner ? min(A + g, C) : c + 1;
#pragma unroll 1
      for (; A < a1; ++A) {
        if (inner && turn++ % shares != share) continue;
        source(A);
      }
    }
  }
  const int t = tb * kWave + lane;
  const bool valid = t < C;
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int l = 0; l <= kFarQ; ++l) {
        if (w == 0) {
          red[l][lane] = make_double2(Lr[l], Li[l]);
        } else {
          const double2 p = red[l][lane];
          red[l][lane] = make_double2(p.x + Lr[l], p.y + Li[l]);
        }
      }
    }
    __syncthreads();
  }
  double2* out = reinterpret_cast<double2*>(wo + (GROUP ? it.lp1 : it.lp0)) +
                 ((size_t)(sp * it.V + v) * 2 + half) * (kFarQ + 1) * C;
  if (valid)
    for (int l = wave; l <= kFarQ; l += 4) out[(size_t)l * C + t] = red[l][lane];
}

// The source shares' sums in a fixed order and in the order of the index:
// forward vectors L_l; backward ones N_m (the transpose, whose result m is
// (-1)^m times the translation's order -m).
__global__ __launch_bounds__(256) void k_far_lsum(FarBlocks B, const double* __restrict__ ro,
                                                  double* __restrict__ wo) {
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  if (far_off(it)) return;
  const int per0 = (it.V * 2 * (kFarQ + 1) * it.P + 255) / 256;
  const bool group = b >= per0;
  if (group) b -= per0;
  const int C = group ? it.C1 : it.P;
  const int ns = group ? it.n1 : it.n0;
  const int e = b * 256 + threadIdx.x;
  if (e >= it.V * 2 * (kFarQ + 1) * C) return;
  const int c = e % C;
  const int l = (e / C) % (kFarQ + 1);
  const int half = (e / (C * (kFarQ + 1))) & 1;
  const int v = e / (C * (kFarQ + 1) * 2);
  const double2* lp = reinterpret_cast<const double2*>(ro + (group ? it.lp1 : it.lp0));
  const size_t stride = (size_t)it.V * 2 * (kFarQ + 1) * C;
  double sr = 0.0, si = 0.0;
#pragma unroll 8
  for (int s = 0; s < ns; ++s) {
    const double2 x = lp[s * stride + e];
    sr += x.x;
    si += x.y;
  }
  double2* ls = reinterpret_cast<double2*>(wo + (group ? it.ls1 : it.ls0)) +
                ((size_t)v * C + c) * kFarW + kFarQ;
  const double s = (l & 1) ? -1.0 : 1.0;
  if (v < it.vf) {
    // forward: half 0 is L_l, half 1 is (-1)^l L_{-l}
    if (half == 0) ls[l] = make_double2(sr, si);
    else if (l > 0) ls[-l] = make_double2(s * sr, s * si);
  } else {
    // backward: N_{-l} = (-1)^l out_l, N_l = (-1)^l out_{-l} = half 1's l
    if (half == 1) ls[l] = make_double2(sr, si);
    else if (l > 0) ls[-l] = make_double2(s * sr, s * si);
  }
}

// ---------------------------------------------------------------------------
// Target side.  A block has 64 consecutive targets of one side, a lane each.
// ---------------------------------------------------------------------------
constexpr int kFarJ = kFarQ + kPMax + 2;   // largest |l - n| is kFarQ + p + 1

struct FarTarget {
  double tx, ty;      // the center (or point)
  double ct, st, R;
  const double* J;    // J_0.. of the center, J'_0.. at nj
  int nj;
  bool pt;
};
// J_n(k R) of any sign of n, 0 past the truncation; a point has J_0 = 1 alone
__device__ __forceinline__ double far_tj(const FarTarget& t, int n, int p) {
  const int a = n < 0 ? -n : n;
  if (a > p) return 0.0;
  const double v = t.pt ? 1.0 : t.J[a];
  return (n < 0 && (a & 1)) ? -v : v;
}
__device__ __forceinline__ double far_tjd(const FarTarget& t, int n, int p) {
  const int a = n < 0 ? -n : n;
  if (a > p || t.pt) return 0.0;
  const double v = t.J[t.nj + a];
  return (n < 0 && (a & 1)) ? -v : v;
}
__device__ __forceinline__ FarTarget far_target(const FarItem& it, const double* ro, int ci) {
  FarTarget t;
  t.pt = it.pt != 0;
  if (t.pt) {
    const double4 g = reinterpret_cast<const double4*>(ro + it.fgeo)[ci];
    t.tx = g.x;
    t.ty = g.y;
    t.ct = 1.0;
    t.st = 0.0;
    t.R = 0.0;
    t.J = nullptr;
    t.nj = 0;
  } else {
    const CenterRec& C = reinterpret_cast<const CenterRec*>(ro + it.ctr)[ci];
    t.tx = C.cx;
    t.ty = C.cy;
    t.ct = C.ct;
    t.st = C.st;
    t.R = C.R;
    t.J = ro + it.jtab + (size_t)ci * it.NJ;
    t.nj = it.NJ / 2;
  }
  return t;
}

__device__ __forceinline__ double2 cpow_int(double2 z, int n) {   // |z| = 1
  double2 b = n < 0 ? conj2(z) : z;
  int a = n < 0 ? -n : n;
  double2 r = make_double2(1.0, 0.0);
  while (a) {
    if (a & 1) r = cmul(r, b);
    b = cmul(b, b);
    a >>= 1;
  }
  return r;
}

// Local expansions to the centers.  MODE 0: per kind the value sum_n a_n W_n,
// W_n = J_n(k R) e^{i n theta}, |n| <= p, into fu[kk][ci].  MODE 1: per kind the sums of
// the target derivatives F_R, F_theta (fu[kk][ci][2]); for points the gradient itself.
// MODE 2: the four center gradients contracted with G over the kinds (fc[ci]): Re of
// K_R, K_theta and grad_v K.  MODE 3: the coefficients themselves, coef[kk][ci][m + p] = a_m,
// |m| <= p.  With tau = |tau| e^{i beta},
//   a_m e^{i m beta} = sum_l (L_l e^{i l beta}) J_{l-m}(k |tau|),
// two real multiply-adds a term: the four waves share the orders m in blocks of kMB,
// whose J_{l-m} slide through registers as l advances.
constexpr int kMB = 6;
template <int MODE>
__global__ __launch_bounds__(256, 2) void k_far_eval(FarBlocks B, const double* __restrict__ ro,
                                                     double* __restrict__ wo,
                                                     double2* __restrict__ coef) {
  __shared__ double Jt[kFarJ + 1][kWave];
  __shared__ double2 LP[kFarW][kWave];
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  if (far_off(it)) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int sides = it.pt ? 1 : it.n_sides;
  const int nb = (it.T + kWave - 1) / kWave;
  const int si = b / nb;
  const int t = (b - si * nb) * kWave + lane;
  const bool valid = t < it.T && si < sides;
  const int tc = valid ? t : it.T - 1;
  const int ci = si * it.T + tc;
  const int m = tc / kQ;
  const int p = it.pt ? 0 : it.p;
  const int pm = MODE == 0 || MODE == 3 ? p : p + 1;   // orders a_m that enter
  const FarTarget tg = far_target(it, ro, ci);
  constexpr int NO = MODE == 0 ? 1 : MODE == 1 ? 2 : 4;
  double2 o[2][2];            // MODE 0, 1: per kind
  double c4[4] = {0, 0, 0, 0};   // MODE 2
  o[0][0] = o[0][1] = o[1][0] = o[1][1] = make_double2(0.0, 0.0);
  const int levels = it.C1 > 0 ? 2 : 1;
  const int nvec = MODE == 2 ? 1 : it.nk;
  const size_t Mt = (size_t)sides * it.T;
  for (int lev = 0; lev < levels; ++lev) {
    const int c = lev ? m / it.g : m;
    const int C = lev ? it.C1 : it.P;
    const FarRec rec = reinterpret_cast<const FarRec*>(ro + (lev ? it.rec1 : it.rec0))[c];
    const double vx = tg.tx - rec.bx, vy = tg.ty - rec.by;
    const double r = sqrt(fma(vx, vx, vy * vy));
    const double2 eb = r > 0.0 ? make_double2(vx / r, vy / r) : make_double2(1.0, 0.0);
    const bool none = far_none(rec);
    __syncthreads();
    if (wave == 0) far_bessel_mem(none ? 0.0 : it.k * r, kFarQ + pm, &Jt[0][lane], kWave);
    const double2 zt = cmul(make_double2(tg.ct, tg.st), conj2(eb));   // e^{i(theta - beta)}
#pragma unroll
    for (int vv = 0; vv < (MODE == 2 ? 1 : 2); ++vv) {
      if (vv >= nvec) break;
      if (vv) __syncthreads();
      // L_l e^{i l beta} of the lane's cluster
      {
        const int l0 = -kFarQ + wave * 13, l1 = min(l0 + 13, kFarQ + 1);
        double2 ph = cpow_int(eb, l0);
        const double2* ls = reinterpret_cast<const double2*>(ro + (lev ? it.ls1 : it.ls0)) +
                            (size_t)c * kFarW + kFarQ;
        const double2* G = reinterpret_cast<const double2*>(ro + it.fG);
        const double2 g0 = MODE == 2 ? G[ci] : make_double2(1.0, 0.0);
        const double2 g1 = MODE == 2 && it.nk > 1 ? G[Mt + ci] : make_double2(0.0, 0.0);
        for (int l = l0; l < l1; ++l) {
          double2 x;
          if (MODE == 2) {
            x = cmul(g0, ls[l]);
            if (it.nk > 1) {
              const double2 y = cmul(g1, ls[(size_t)C * kFarW + l]);
              x = make_double2(x.x + y.x, x.y + y.y);
            }
          } else {
            x = ls[(size_t)vv * C * kFarW + l];
          }
          LP[l + kFarQ][lane] = none ? make_double2(0.0, 0.0) : cmul(x, ph);
          ph = cmul(ph, eb);
        }
      }
      __syncthreads();
      const int nblk = (2 * pm + 1 + kMB - 1) / kMB;
#pragma unroll 1
      for (int blk = wave; blk < nblk; blk += 4) {
        const int m0 = -pm + blk * kMB;
        double ar[kMB], ai[kMB], w[kMB];
#pragma unroll
        for (int i = 0; i < kMB; ++i) ar[i] = ai[i] = 0.0;
        auto jt = [&](int d) {
          const int a = d < 0 ? -d : d;
          const double v = a <= kFarQ + pm ? Jt[a][lane] : 0.0;
          return (d < 0 && (a & 1)) ? -v : v;
        };
        // w[i] = J_{l - m0 - i}
#pragma unroll
        for (int i = 0; i < kMB; ++i) w[i] = jt(-kFarQ - 1 - m0 - i);
#pragma unroll 1
        for (int l = -kFarQ; l <= kFarQ; l += 7) {
#pragma unroll
          for (int u = 0; u < 7; ++u) {
#pragma unroll
            for (int i = kMB - 1; i > 0; --i) w[i] = w[i - 1];
            w[0] = jt(l + u - m0);
            const double2 x = LP[l + u + kFarQ][lane];
#pragma unroll
            for (int i = 0; i < kMB; ++i) {
              ar[i] = fma(x.x, w[i], ar[i]);
              ai[i] = fma(x.y, w[i], ai[i]);
            }
          }
        }
        const double2 zs = MODE == 3 ? conj2(eb) : zt;
        double2 zp = cpow_int(zs, m0);
#pragma unroll
        for (int i = 0; i < kMB; ++i) {
          const int mm = m0 + i;
          if (MODE == 3) {
            if (mm <= pm && valid) {
              const double2 a = cmul(make_double2(ar[i], ai[i]), zp);   // a_m
              double2* q = coef + ((size_t)vv * Mt + ci) * (2 * p + 1) + mm + p;
              const double2 f = lev ? *q : make_double2(0.0, 0.0);
              *q = make_double2(f.x + a.x, f.y + a.y);
            }
          } else if (mm <= pm) {
            const double2 a = cmul(make_double2(ar[i], ai[i]), zp);   // a_m e^{i m theta}
            const double jm = far_tj(tg, mm, p);
            if (MODE == 0) {
              o[vv][0].x = fma(a.x, jm, o[vv][0].x);
              o[vv][0].y = fma(a.y, jm, o[vv][0].y);
            } else if (MODE == 1 && !tg.pt) {
              const double jd = it.k * far_tjd(tg, mm, p), jt2 = mm * jm;
              o[vv][0].x = fma(a.x, jd, o[vv][0].x);
              o[vv][0].y = fma(a.y, jd, o[vv][0].y);
              o[vv][1].x = fma(-a.y, jt2, o[vv][1].x);
              o[vv][1].y = fma(a.x, jt2, o[vv][1].y);
            } else {
              // s1, s2 of the shift of the center: a_m W_{m-1}, a_m W_{m+1}
              const double2 eth = make_double2(tg.ct, tg.st);
              const double j1 = far_tj(tg, mm - 1, p), j2 = far_tj(tg, mm + 1, p);
              const double2 s1 = cmul(make_double2(a.x * j1, a.y * j1), conj2(eth));
              const double2 s2 = cmul(make_double2(a.x * j2, a.y * j2), eth);
              const double hk = 0.5 * it.k;
              // d/dc_x = (k/2)(s1 - s2), d/dc_y = (i k/2)(s1 + s2)
              const double2 gx = make_double2(hk * (s1.x - s2.x), hk * (s1.y - s2.y));
              const double2 gy = make_double2(-hk * (s1.y + s2.y), hk * (s1.x + s2.x));
              if (MODE == 1) {
                o[vv][0].x += gx.x;
                o[vv][0].y += gx.y;
                o[vv][1].x += gy.x;
                o[vv][1].y += gy.y;
              } else {
                c4[0] = fma(a.x, it.k * far_tjd(tg, mm, p), c4[0]);
                c4[1] = fma(-a.y, mm * jm, c4[1]);
                c4[2] -= gx.x;   // grad_v = -grad_c
                c4[3] -= gy.x;
              }
            }
          }
          zp = cmul(zp, zs);
        }
      }
    }
  }
  if (MODE == 3) return;
  // add the four waves (in wave order) through LDS
  __syncthreads();
  double* red = &LP[0][0].x;   // [4][8][64]
  const int nd = MODE == 2 ? 4 : it.nk * NO * 2;
  {
    double v[8];
    if (MODE == 2) {
      for (int i = 0; i < 4; ++i) v[i] = c4[i];
    } else {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          if (q < NO) {
            v[(kk * NO + q) * 2] = o[kk][q].x;
            v[(kk * NO + q) * 2 + 1] = o[kk][q].y;
          }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < nd) red[(wave * 8 + i) * kWave + lane] = v[i];
  }
  __syncthreads();
  if (valid) {
    for (int i = wave; i < nd; i += 4) {
      const double s = ((red[i * kWave + lane] + red[(8 + i) * kWave + lane]) +
                        red[(16 + i) * kWave + lane]) + red[(24 + i) * kWave + lane];
      if (MODE == 2) {
        wo[it.fc + (size_t)ci * 4 + i] = s;
      } else {
        const int kk = i / (2 * NO), q = i % (2 * NO);
        wo[it.fu + ((size_t)kk * Mt + ci) * 2 * NO + q] = s;
      }
    }
  }
}

// Adjoint, target side: T_l = sum_c G_c E_l(c) per kind,
// E_l = e^{i l beta} sum_m (W_m e^{-i m beta}) J_{l-m}(k|tau|), over the block's targets of
// each panel (16 lanes) and of the group (64: four panels, a group or half of one).
// tp0[si][kk][panel], tp1[si (g / 4) + half][kk][group].
__global__ __launch_bounds__(256) void k_far_t(FarBlocks B, const double* __restrict__ ro,
                                               double* __restrict__ wo) {
  __shared__ double Jt[kFarJ + 1][kWave];
  __shared__ double2 Wm[2 * kPMax + 1][kWave];
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  if (far_off(it)) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int sides = it.pt ? 1 : it.n_sides;
  const int nb = (it.T + kWave - 1) / kWave;
  const int si = b / nb;
  const int tb = b - si * nb;
  const int t = tb * kWave + lane;
  const bool valid = t < it.T;
  const int tc = valid ? t : it.T - 1;
  const int ci = si * it.T + tc;
  const int m = tc / kQ;
  const int p = it.pt ? 0 : it.p;
  const FarTarget tg = far_target(it, ro, ci);
  const size_t Mt = (size_t)sides * it.T;
  const double2* G = reinterpret_cast<const double2*>(ro + it.fG);
  double2 g[2];
  g[0] = valid ? G[ci] : make_double2(0.0, 0.0);
  g[1] = valid && it.nk > 1 ? G[Mt + ci] : make_double2(0.0, 0.0);
  const int levels = it.C1 > 0 ? 2 : 1;
  for (int lev = 0; lev < levels; ++lev) {
    const int c = lev ? m / it.g : m;
    const int C = lev ? it.C1 : it.P;
    const FarRec rec = reinterpret_cast<const FarRec*>(ro + (lev ? it.rec1 : it.rec0))[c];
    const double vx = tg.tx - rec.bx, vy = tg.ty - rec.by;
    const double r = sqrt(fma(vx, vx, vy * vy));
    const double2 eb = r > 0.0 ? make_double2(vx / r, vy / r) : make_double2(1.0, 0.0);
    const bool none = far_none(rec);
    __syncthreads();
    if (wave == 0) far_bessel_mem(none ? 0.0 : it.k * r, kFarQ + p, &Jt[0][lane], kWave);
    const double2 zt = cmul(make_double2(tg.ct, tg.st), conj2(eb));
    if (wave > 0) {   // W_m e^{-i m beta}, the orders shared by three waves
      const int per = (2 * p + 3) / 3;
      const int a0 = (wave - 1) * per, a1 = min(a0 + per, 2 * p + 1);
      double2 zp = cpow_int(zt, a0 - p);
      for (int a = a0; a < a1; ++a) {
        const double j = far_tj(tg, a - p, p);
        Wm[a][lane] = make_double2(zp.x * j, zp.y * j);
        zp = cmul(zp, zt);
      }
    }
    __syncthreads();
    double2* tp = reinterpret_cast<double2*>(wo + (lev ? it.tp1 : it.tp0));
    for (int l0 = -kFarQ + wave * 7; l0 <= kFarQ; l0 += 28) {   // 7 blocks of 7 orders
      double ar[7], ai[7], w[7];
      auto jt = [&](int d) {
        const int a = d < 0 ? -d : d;
        const double v = a <= kFarQ + p ? Jt[a][lane] : 0.0;
        return (d < 0 && (a & 1)) ? -v : v;
      };
      // w[i] = J_{l0 + i - m}; as m grows the window slides down
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        ar[i] = ai[i] = 0.0;
        w[i] = jt(l0 + i + p + 1);
      }
      for (int mm = -p; mm <= p; ++mm) {
#pragma unroll
        for (int i = 6; i > 0; --i) w[i] = w[i - 1];
        w[0] = jt(l0 - mm);
        const double2 x = Wm[mm + p][lane];
#pragma unroll
        for (int i = 0; i < 7; ++i) {
          ar[i] = fma(x.x, w[i], ar[i]);
          ai[i] = fma(x.y, w[i], ai[i]);
        }
      }
      double2 ph = cpow_int(eb, l0);
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        const double2 E = cmul(make_double2(ar[i], ai[i]), ph);
        ph = cmul(ph, eb);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          if (kk >= it.nk) break;
          double2 s = cmul(g[kk], E);
          if (none) s = make_double2(0.0, 0.0);
          const int top = lev ? 64 : 16;
#pragma unroll
          for (int off = 1; off < 64; off <<= 1)
            if (off < top) {
              s.x += __shfl_xor(s.x, off);
              s.y += __shfl_xor(s.y, off);
            }
          if (lev == 0) {
            if ((lane & 15) == 0 && valid)
              tp[(((size_t)si * it.nk + kk) * C + c) * kFarW + l0 + i + kFarQ] = s;
          } else if (lane == 0) {
            tp[(((size_t)(si * (it.g / 4) + tb % (it.g / 4)) * it.nk + kk) * C + c) * kFarW + l0 + i + kFarQ] = s;
          }
        }
      }
    }
  }
}

// T's parts added, in the rows of the translation: row 0 (-1)^m T_{-m}, row 1 T_m
__global__ __launch_bounds__(256) void k_far_rows(FarBlocks B, const double* __restrict__ ro,
                                                  double* __restrict__ wo) {
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  if (far_off(it)) return;
  const int per0 = (it.nk * it.P * kFarW + 255) / 256;
  const bool group = b >= per0;
  if (group) b -= per0;
  const int C = group ? it.C1 : it.P;
  const int e = b * 256 + threadIdx.x;
  if (e >= it.nk * C * kFarW) return;
  const int m = e % kFarW - kFarQ;
  const int c = (e / kFarW) % C;
  const int kk = e / (kFarW * C);
  const double2* tp = reinterpret_cast<const double2*>(ro + (group ? it.tp1 : it.tp0));
  const int sides = it.pt ? 1 : it.n_sides;
  double2 s = make_double2(0.0, 0.0);
  for (int si = 0; si < sides; ++si)
    for (int h = 0; h < (group ? it.g / 4 : 1); ++h) {
      // the last group's second block is missing when it has at most four panels
      if (group && c * it.g + 4 * h >= it.P) continue;
      const int part = group ? si * (it.g / 4) + h : si;
      const double2 x = tp[(((size_t)part * it.nk + kk) * C + c) * kFarW + m + kFarQ];
      s.x += x.x;
      s.y += x.y;
    }
  double2* rows = reinterpret_cast<double2*>(wo + (group ? it.rows1 : it.rows0));
  const int v = it.vf + kk;
  const double sg = (m & 1) ? -1.0 : 1.0;
  rows[((size_t)(v * 2 + 0) * C + c) * kFarW + kFarQ - m] = make_double2(sg * s.x, sg * s.y);
  rows[((size_t)(v * 2 + 1) * C + c) * kFarW + kFarQ + m] = s;
}

// Adjoint, source side: per far source the field of the far targets' weights and its
// derivatives.  With the shifted sums P_s = sum_m N_{m+s} g_m (g_m = J_m e^{-i m alpha}),
// d/dnu = conj(nu) A + nu B with A = (k/2) P_1, B = -(k/2) P_{-1}, A A = (k^2/4) P_2,
// B B = (k^2/4) P_{-2}, A B = -(k^2/4) P_0.  fs[kk]: conj of the density gradient's sum;
// fs[nk]: position; fs[nk + 1]: for a layer potential's sources the angle sum Re(q dK/dpsi),
// for the split's far sources (pt) the normal's gradient.
__global__ __launch_bounds__(64) void k_far_src(FarBlocks B, const double* __restrict__ ro,
                                                double* __restrict__ wo, int geom) {
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  if (far_off(it)) return;
  const int lane = threadIdx.x;
  const int per = (it.fqs + kWave - 1) / kWave;
  const int m = b / per;
  const int s0 = (b - m * per) * kWave;
  const bool valid = s0 + lane < it.fqs;
  const int j = m * it.fqs + (valid ? s0 + lane : it.fqs - 1);
  const size_t Nf = (size_t)it.P * it.fqs;
  const double4 g = reinterpret_cast<const double4*>(ro + it.fgeo)[j];
  const double2* dens = reinterpret_cast<const double2*>(ro + it.fdens);
  const int nk = it.nk;
  // sums P_s, s = -2..2, per kind (the single layer needs |s| <= 1)
  double2 P[2][5];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int s = 0; s < 5; ++s) P[a][s] = make_double2(0.0, 0.0);
  const int levels = it.C1 > 0 ? 2 : 1;
  for (int lev = 0; lev < levels; ++lev) {
    const int c = lev ? m / it.g : m;
    const int C = lev ? it.C1 : it.P;
    const FarRec rec = reinterpret_cast<const FarRec*>(ro + (lev ? it.rec1 : it.rec0))[c];
    if (far_none(rec)) continue;
    const double vx = g.x - rec.bx, vy = g.y - rec.by;
    const double r = sqrt(fma(vx, vx, vy * vy));
    const double2 e = r > 0.0 ? make_double2(vx / r, -vy / r) : make_double2(1.0, 0.0);
    double J[kFarQ + 3];
    far_bessel<kFarQ + 2>(it.k * r, J);
    // N of this cluster (wave-uniform), zero past +-kFarQ
    const double2* __restrict__ N0 =
        reinterpret_cast<const double2*>(ro + (lev ? it.ls1 : it.ls0)) +
        ((size_t)it.vf * C + c) * kFarW + kFarQ;
    auto add = [&](const double2* __restrict__ N, double2 (&Q)[5], int mm, double2 gm) {
#pragma unroll
      for (int s = -2; s <= 2; ++s) {
        if (mm + s < -kFarQ || mm + s > kFarQ) continue;
        const double2 n = N[mm + s];
        Q[s + 2].x = fma(n.x, gm.x, fma(-n.y, gm.y, Q[s + 2].x));
        Q[s + 2].y = fma(n.x, gm.y, fma(n.y, gm.x, Q[s + 2].y));
      }
    };
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (kk >= nk) break;
      const double2* __restrict__ N = N0 + (size_t)kk * C * kFarW;
      double2 Q[5];
#pragma unroll
      for (int s = 0; s < 5; ++s) Q[s] = make_double2(0.0, 0.0);
      double2 em = make_double2(1.0, 0.0);
#pragma unroll
      for (int mm = 0; mm <= kFarQ + 2; ++mm) {
        const double2 gm = make_double2(J[mm] * em.x, J[mm] * em.y);
        // the row is read again for every order, one order in flight
        const double2* __restrict__ Nm = N + opaque_zero();
        add(Nm, Q, mm, gm);
        if (mm > 0) {
          const double s = (mm & 1) ? -1.0 : 1.0;
          add(Nm, Q, -mm, make_double2(s * gm.x, -s * gm.y));
        }
        em = cmul(em, e);
        asm volatile("" : "+v"(em.x), "+v"(em.y));
#pragma unroll
        for (int s = 0; s < 5; ++s) asm volatile("" : "+v"(Q[s].x), "+v"(Q[s].y));
      }
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        P[kk][s].x += Q[s].x;
        P[kk][s].y += Q[s].y;
      }
    }
  }
  if (!valid) return;
  double2* fs = reinterpret_cast<double2*>(wo + it.fs);
  const double hk = 0.5 * it.k;
  const double2 nu = make_double2(g.z, g.w), nc = conj2(nu);
  double gx = 0.0, gy = 0.0, gp = 0.0, gnx = 0.0, gny = 0.0;
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    if (kk >= nk) break;
    const bool dbl = it.kind == 2 || kk == 1;
    const double2 q = dens[(size_t)kk * Nf + j];
    const double2 p0 = P[kk][2];
    const double2 A = make_double2(hk * P[kk][3].x, hk * P[kk][3].y);
    const double2 Bm = make_double2(-hk * P[kk][1].x, -hk * P[kk][1].y);
    double2 val, px, py;
    if (!dbl) {
      val = p0;
      px = make_double2(A.x + Bm.x, A.y + Bm.y);          // d/dx = A + B
      py = make_double2(A.y - Bm.y, Bm.x - A.x);          // d/dy = -i A + i B
    } else {
      const double2 va = cmul(nc, A), vb = cmul(nu, Bm);
      val = make_double2(va.x + vb.x, va.y + vb.y);
      const double h2 = hk * hk;
      const double2 AA = make_double2(h2 * P[kk][4].x, h2 * P[kk][4].y);
      const double2 BB = make_double2(h2 * P[kk][0].x, h2 * P[kk][0].y);
      const double2 AB = make_double2(-h2 * p0.x, -h2 * p0.y);
      // A(d/dnu) = conj(nu) AA + nu AB, B(d/dnu) = conj(nu) AB + nu BB
      const double2 a1 = cmul(nc, AA), a2 = cmul(nu, AB), b1 = cmul(nc, AB), b2 = cmul(nu, BB);
      const double2 dA = make_double2(a1.x + a2.x, a1.y + a2.y);
      const double2 dB = make_double2(b1.x + b2.x, b1.y + b2.y);
      px = make_double2(dA.x + dB.x, dA.y + dB.y);
      py = make_double2(dA.y - dB.y, dB.x - dA.x);
      // d/dpsi = -d/d(arg nu): i conj(nu) A - i nu B
      const double2 dp = make_double2(-(va.y - vb.y), va.x - vb.x);
      gp += q.x * dp.x - q.y * dp.y;
      // gradient in nu itself: d/dx, d/dy of the field
      const double2 nx = make_double2(A.x + Bm.x, A.y + Bm.y);
      const double2 ny = make_double2(A.y - Bm.y, Bm.x - A.x);
      gnx += q.x * nx.x - q.y * nx.y;
      gny += q.x * ny.x - q.y * ny.y;
    }
    // the pair passes keep conj(sum G K) for a layer potential's sources, the sum itself
    // for the split's
    fs[(size_t)kk * Nf + j] = it.pt ? val : conj2(val);
    gx += q.x * px.x - q.y * px.y;
    gy += q.x * py.x - q.y * py.y;
  }
  if (geom) {
    fs[(size_t)nk * Nf + j] = make_double2(gx, gy);
    fs[(size_t)(nk + 1) * Nf + j] = it.pt ? make_double2(gnx, gny) : make_double2(gp, 0.0);
  }
}

// Lists of the panels that no expansion takes: one wave per panel scans all panels (64 per
// ballot) and writes them in ascending order, at most kNearCap, and their count.
__global__ __launch_bounds__(256) void k_far_lists(FarBlocks B, const double* __restrict__ ro,
                                                   double* __restrict__ wo) {
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int m = b * 4 + wave;
  if (m >= it.P) return;
  FarRel R;
  R.r0 = reinterpret_cast<const FarRec*>(ro + it.rec0);
  R.r1 = it.C1 > 0 ? reinterpret_cast<const FarRec*>(ro + it.rec1) : nullptr;
  R.g = it.g;
  R.bnd = it.pt ? reinterpret_cast<const double4*>(ro + it.bnd) : nullptr;
  R.g2 = it.g2;
  int* count = reinterpret_cast<int*>(wo + it.mcount);
  int* list = reinterpret_cast<int*>(wo + it.mlist);
  int n = 0;
  for (int w0 = 0; w0 < it.P; w0 += kWave) {
    const int mp = w0 + lane;
    const bool nr = mp < it.P && !far_panels(R, m, mp);
    const unsigned long long mask = __ballot(nr);
    const int pos = n + __popcll(mask & ((1ULL << lane) - 1ULL));
    if (nr && pos < kNearCap) list[(size_t)m * kNearCap + pos] = mp;
    n += __popcll(mask);
  }
  if (lane == 0) {
    count[m] = n;
    if (far_heavy(n, it.P))
      atomicAdd(const_cast<unsigned long long*>(&it.heavy), (unsigned long long)n);
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_near_1(NearPass, int, const FarBlocks&, int, double*, double*, hipStream_t);
hipError_t launch_near_2(NearPass, int, const FarBlocks&, int, double*, double*, hipStream_t);
hipError_t launch_near_3(NearPass, int, const FarBlocks&, int, double*, double*, hipStream_t);

hipError_t launch_near(NearPass pass, int p, int kind, const FarBlocks& B, int blocks,
                       double* ws, double* out, hipStream_t s) {
  return kind == 1   ? launch_near_1(pass, p, B, blocks, ws, out, s)
         : kind == 2 ? launch_near_2(pass, p, B, blocks, ws, out, s)
                     : launch_near_3(pass, p, B, blocks, ws, out, s);
}

hipError_t launch_tiles_1(int, FarItem*, int, int, double*, hipStream_t);
hipError_t launch_tiles_2(int, FarItem*, int, int, double*, hipStream_t);
hipError_t launch_tiles_3(int, FarItem*, int, int, double*, hipStream_t);

hipError_t launch_near_tiles(int p, int kind, FarItem* items, int n, int blocks, double* ws,
                             hipStream_t s) {
  return kind == 1   ? launch_tiles_1(p, items, n, blocks, ws, s)
         : kind == 2 ? launch_tiles_2(p, items, n, blocks, ws, s)
                     : launch_tiles_3(p, items, n, blocks, ws, s);
}

int far_blocks(const FarItem& it, FarStep step) {
  const int sides = it.pt ? 1 : it.n_sides;
  switch (step) {
    case kStepClusters: return it.P + it.C1;
    case kStepM2L: return 2 * it.V * ((it.P + kWave - 1) / kWave) * it.n0;
    case kStepM2LGroups: return 2 * it.V * ((it.C1 + kWave - 1) / kWave) * it.n1;
    case kStepSum:
      return (it.V * 2 * (kFarQ + 1) * it.P + 255) / 256 +
             (it.V * 2 * (kFarQ + 1) * it.C1 + 255) / 256;
    case kStepTargets: return sides * ((it.T + kWave - 1) / kWave);
    case kStepRows:
      return (it.nk * it.P * kFarW + 255) / 256 + (it.nk * it.C1 * kFarW + 255) / 256;
    case kStepSources: return it.P * ((it.fqs + kWave - 1) / kWave);
    case kStepLists: return (it.P + 3) / 4;
    case kStepCenters: return (it.Mc + 3) / 4;
    case kStepNear: return it.quad ? it.Mc : (it.Mc + 3) / 4;
    case kStepChunks: return (it.P * near_subs(it.qs) * it.nsrc + 3) / 4;
    case kStepCenterSums: return (it.Mc + 63) / 64;
  }
  return 0;
}

hipError_t launch_far_recs(const FarBlocks& B, int blocks, const double* nodes, double* ws,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_far_recs, dim3(blocks), dim3(64), 0, s, B, ws, nodes, ws);
  return hipGetLastError();
}
hipError_t launch_far_lists(const FarBlocks& B, int blocks, double* ws, hipStream_t s) {
  hipLaunchKernelGGL(k_far_lists, dim3(blocks), dim3(256), 0, s, B, ws, ws);
  return hipGetLastError();
}
hipError_t launch_far_p2m(const FarBlocks& B, int blocks, double* ws, hipStream_t s) {
  hipLaunchKernelGGL(k_far_p2m, dim3(blocks), dim3(64), 0, s, B, ws, ws);
  return hipGetLastError();
}
hipError_t launch_far_m2l(bool groups, const FarBlocks& B, int blocks, double* ws,
                          hipStream_t s) {
  if (groups)
    hipLaunchKernelGGL(k_far_m2l<true>, dim3(blocks), dim3(256), 0, s, B, ws, ws);
  else
    hipLaunchKernelGGL(k_far_m2l<false>, dim3(blocks), dim3(256), 0, s, B, ws, ws);
  return hipGetLastError();
}
hipError_t launch_far_lsum(const FarBlocks& B, int blocks, double* ws, hipStream_t s) {
  hipLaunchKernelGGL(k_far_lsum, dim3(blocks), dim3(256), 0, s, B, ws, ws);
  return hipGetLastError();
}
hipError_t launch_far_eval(int mode, const FarBlocks& B, int blocks, double* ws, double2* coef,
                           hipStream_t s) {
  const dim3 grid(blocks), block(256);
  if (mode == 0)
    hipLaunchKernelGGL(k_far_eval<0>, grid, block, 0, s, B, ws, ws, coef);
  else if (mode == 1)
    hipLaunchKernelGGL(k_far_eval<1>, grid, block, 0, s, B, ws, ws, coef);
  else if (mode == 2)
    hipLaunchKernelGGL(k_far_eval<2>, grid, block, 0, s, B, ws, ws, coef);
  else
    hipLaunchKernelGGL(k_far_eval<3>, grid, block, 0, s, B, ws, ws, coef);
  return hipGetLastError();
}
hipError_t launch_far_t(const FarBlocks& B, int blocks, double* ws, hipStream_t s) {
  hipLaunchKernelGGL(k_far_t, dim3(blocks), dim3(256), 0, s, B, ws, ws);
  return hipGetLastError();
}
hipError_t launch_far_rows(const FarBlocks& B, int blocks, double* ws, hipStream_t s) {
  hipLaunchKernelGGL(k_far_rows, dim3(blocks), dim3(256), 0, s, B, ws, ws);
  return hipGetLastError();
}
hipError_t launch_far_src(const FarBlocks& B, int blocks, double* ws, bool geom, hipStream_t s) {
  hipLaunchKernelGGL(k_far_src, dim3(blocks), dim3(64), 0, s, B, ws, ws, geom ? 1 : 0);
  return hipGetLastError();
}

FarPlan far_single(const FarItem& it, const FarItem* dev) {
  FarPlan P;
  for (int i = 0; i <= kStepLists; ++i) {
    P.at[i] = FarBlocks{dev, nullptr, 1};
    P.blocks[i] = far_blocks(it, (FarStep)i);
  }
  return P;
}

void far_shape(FarItem* it, bool fwd, bool bwd) {
  it->vf = fwd ? it->nk : 0;
  it->V = it->vf + (bwd ? it->nk : 0);
  it->n0 = far_share(it->P, it->V, it->m2l_blocks, it->C1 > 0);
  it->n1 = it->C1 ? far_share(it->C1, it->V, it->m2l_blocks, false) : 1;
  it->off_pairs = (!(fwd && bwd)                      ? kFarOffPass
                   : it->P <= kNearSlotsSmallPanels ? kFarOffAdjointSmall
                                                    : kFarOffAdjoint) *
                  it->P * it->P;
}

hipError_t far_fields(const FarPlan& P, const double* nodes, double* ws, bool fwd, bool bwd,
                      int eval, bool src, bool geom, bool lists, hipStream_t s, double2* coef) {
  hipError_t e = launch_far_recs(P.at[kStepClusters], P.blocks[kStepClusters], nodes, ws, s);
  if (e == hipSuccess && lists) e = launch_far_lists(P.at[kStepLists], P.blocks[kStepLists], ws, s);
  if (e == hipSuccess && fwd)
    e = launch_far_p2m(P.at[kStepClusters], P.blocks[kStepClusters], ws, s);
  if (e == hipSuccess && bwd) e = launch_far_t(P.at[kStepTargets], P.blocks[kStepTargets], ws, s);
  if (e == hipSuccess && bwd) e = launch_far_rows(P.at[kStepRows], P.blocks[kStepRows], ws, s);
  if (e == hipSuccess) e = launch_far_m2l(false, P.at[kStepM2L], P.blocks[kStepM2L], ws, s);
  if (e == hipSuccess && P.blocks[kStepM2LGroups] > 0)
    e = launch_far_m2l(true, P.at[kStepM2LGroups], P.blocks[kStepM2LGroups], ws, s);
  if (e == hipSuccess) e = launch_far_lsum(P.at[kStepSum], P.blocks[kStepSum], ws, s);
  if (e == hipSuccess && eval >= 0)
    e = launch_far_eval(eval, P.at[kStepTargets], P.blocks[kStepTargets], ws, coef, s);
  if (e == hipSuccess && src)
    e = launch_far_src(P.at[kStepSources], P.blocks[kStepSources], ws, geom, s);
  return e;
}

}  // namespace qbx
