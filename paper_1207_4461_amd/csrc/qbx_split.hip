// Near/far split of the forward (Section 5: QBX only for the panels near a
// target, direct evaluation by the smooth source rule for all others).
//
// Near relation.  Per panel, b_m is the mean of its 16 nodes (added in node
// order, then times 1/16) and rad2_m = max_a |X_{m,a} - b_m|^2.  Source panel m'
// is near target panel m when
//     |b_m - b_m'|^2 < gamma^2 max(rad2_m, rad2_m').
// Every product and sum of the test is rounded on its own (contraction off), so
// the near pass, the far pass and any IEEE double evaluation of the same formula
// take the same decisions.  A panel is always near itself (gamma > 0).
//
// Near pass (k_near_forward of qbx_near.hip): one wave per center over the sources of
// its panel's near list.  Far pairs: from 96 panels on through panel expansions
// (qbx_far.hip), and the few that none reaches by k_split_mid; below that, and where none
// reaches many (far_off), by k_split_far: the 64 lanes are 64 consecutive targets and the
// sources of a run of panels are wave-uniform (scalar loads); a far pair adds
//     S: w sigma H_0(k rho),    D: w mu k H_1(k rho) (x - x').n' / rho,
// rho = |x - x'|, the normal derivative of H_0(k|x - x'|) at the source (the
// seeds from the shortest fits when every lane of the wave has k rho >= 60).  These
// sums do not depend on the side, so both sides share one far pass.  The
// finalize adds, per center, the near sum and the far sums of its target in a
// fixed order and applies i/4.
#include <type_traits>

#include "qbx_far.h"
#include "qbx_pair.h"
#include "qbx_panel.h"

namespace qbx {


// Near lists: one wave per panel m scans all panels (64 per ballot) and writes
// the near ones in ascending order, at most kNearCap of them, and their count.
__global__ __launch_bounds__(256) void k_near_lists(int NP, const double4* __restrict__ bnd,
                                                    double g2, int* __restrict__ count,
                                                    int* __restrict__ list) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int m = blockIdx.x * 4 + wave;
  if (m >= NP) return;
  const double4 bm = bnd[m];
  int n = 0;
  for (int w0 = 0; w0 < NP; w0 += kWave) {
    const int mp = w0 + lane;
    const bool nr = mp < NP && panels_near(bm, bnd[mp], g2);
    const unsigned long long mask = __ballot(nr);
    const int pos = n + __popcll(mask & ((1ULL << lane) - 1ULL));
    if (nr && pos < kNearCap) list[(size_t)m * kNearCap + pos] = mp;
    n += __popcll(mask);
  }
  if (lane == 0) count[m] = n;
}

// the panel's record {b_x, b_y, rad2, sqrt(rad2)} from its nodes
__device__ __forceinline__ double4 panel_bounds(const double* __restrict__ X) {
#pragma clang fp contract(off)
  double sx = X[0], sy = X[1];
  for (int a = 1; a < kQ; ++a) {
    sx = sx + X[2 * a];
    sy = sy + X[2 * a + 1];
  }
  const double bx = sx * 0.0625, by = sy * 0.0625;
  double r2 = 0.0;
  for (int a = 0; a < kQ; ++a) {
    const double dx = X[2 * a] - bx;
    const double dy = X[2 * a + 1] - by;
    r2 = fmax(r2, dx * dx + dy * dy);
  }
  // .w: the node radius, which bounds |x - x'| from below for a whole panel of
  // the far sources (the panel's nodes) at once
  return make_double4(bx, by, r2, sqrt(r2));
}

// The panels' records (one thread of each panel's; a launch of their own took as long as this
// one) and the Nystrom grid as the far sources (one thread per node t = 16 m + a): the node
// itself, the outward normal n = (y', -x')/|X'| from the 16-node derivative (the
// table's Dn rows, as for the centers), the 16-point Gauss-Legendre weight
// w = omega_a |X'(tau_a)| (the table's w16) and the weighted node densities w sigma.
__global__ __launch_bounds__(256) void k_nystrom_sources(int T, int nk,
                                                         const double* __restrict__ nodes,
                                                         const double* __restrict__ density,
                                                         const double* __restrict__ Dn,
                                                         const double* __restrict__ w16,
                                                         double4* __restrict__ bnd,
                                                         double4* __restrict__ ngeo,
                                                         double2* __restrict__ ndens,
                                                         double* __restrict__ nw) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const int m = t / kQ, a = t - m * kQ;
  const double* X = nodes + (size_t)m * 2 * kQ;
  if (a == 0) bnd[m] = panel_bounds(X);
  const double* Dr = Dn + a * kQ;
  double tx = 0.0, ty = 0.0;
  for (int c = 0; c < kQ; ++c) {
    tx = fma(Dr[c], X[2 * c], tx);
    ty = fma(Dr[c], X[2 * c + 1], ty);
  }
  const double sp = sqrt(tx * tx + ty * ty);
  const double inv = 1.0 / sp;
  const double w = w16[a] * sp;
  ngeo[t] = make_double4(X[2 * a], X[2 * a + 1], ty * inv, -tx * inv);
  nw[t] = w;
  for (int kk = 0; kk < nk; ++kk) {
    const double* sg = density + 2 * ((size_t)kk * T + t);
    ndens[(size_t)kk * T + t] = make_double2(w * sg[0], w * sg[1]);
  }
}

// one far pair: w sigma H_0 (S) and w mu H_1 (x - x').n' / rho (D; the factor k is
// applied once per sum), with the pair's weighted densities wS (S) and wD (D)
template <bool kS, bool kD>
__device__ __forceinline__ void far_accumulate_q(const double2& wS, const double2& wD,
                                                 const double4& g, double dx, double dy,
                                                 double ir, const H01& h, double& sr, double& si,
                                                 double& dr, double& di) {
  if (kS) {
    sr = fma(wS.x, h.h0r, fma(-wS.y, h.h0i, sr));
    si = fma(wS.x, h.h0i, fma(wS.y, h.h0r, si));
  }
  if (kD) {
    const double f = fma(dx, g.z, dy * g.w) * ir;   // (x - x').n' / rho
    const double wr = wD.x * f, wi = wD.y * f;
    dr = fma(wr, h.h1r, fma(-wi, h.h1i, dr));
    di = fma(wr, h.h1i, fma(wi, h.h1r, di));
  }
}

// one far pair of the target derivatives: the gradient's sums (x, y; complex), without
// the factors -k (S) and k (D)
template <bool kS, bool kD>
__device__ __forceinline__ void grad_accumulate(const double2& wS, const double2& wD,
                                                const double4& g, double dx, double dy, double ir,
                                                double k, const H01& h, double (&S)[4],
                                                double (&D)[4]) {
  const double ux = dx * ir, uy = dy * ir;
  if (kS) {
    const double hr = fma(wS.x, h.h1r, -wS.y * h.h1i), hi = fma(wS.x, h.h1i, wS.y * h.h1r);
    S[0] = fma(hr, ux, S[0]);
    S[1] = fma(hi, ux, S[1]);
    S[2] = fma(hr, uy, S[2]);
    S[3] = fma(hi, uy, S[3]);
  }
  if (kD) {
    const double f = fma(ux, g.z, uy * g.w);
    // k H_0 f u + (H_1 / rho)(n' - 2 f u), times w mu
    const double a_r = k * f * h.h0r, a_i = k * f * h.h0i;
    const double b_r = h.h1r * ir, b_i = h.h1i * ir;
    const double vx = fma(-2.0 * f, ux, g.z), vy = fma(-2.0 * f, uy, g.w);
    const double cxr = fma(a_r, ux, b_r * vx), cxi = fma(a_i, ux, b_i * vx);
    const double cyr = fma(a_r, uy, b_r * vy), cyi = fma(a_i, uy, b_i * vy);
    D[0] = fma(wD.x, cxr, fma(-wD.y, cxi, D[0]));
    D[1] = fma(wD.x, cxi, fma(wD.y, cxr, D[1]));
    D[2] = fma(wD.x, cyr, fma(-wD.y, cyi, D[2]));
    D[3] = fma(wD.x, cyi, fma(wD.y, cyr, D[3]));
  }
}

// one far pair of the adjoint, source side: the cotangent weights GS, GD of the target
// times H_0 (S) and H_1 (x - x').n' / rho (D) into v; GEO: the gradients for the
// source's position and normal, contracted with its weighted densities, into e (without
// the factor k)
template <bool kS, bool kD, bool GEO>
__device__ __forceinline__ void adj_accumulate(const double2& GS, const double2& GD,
                                               const double2& qS, const double2& qD,
                                               const double4& g, double dx, double dy, double ir,
                                               double k, const H01& h, double (&v)[4],
                                               double (&e)[4]) {
  if (kS) {
    v[0] = fma(GS.x, h.h0r, fma(-GS.y, h.h0i, v[0]));
    v[1] = fma(GS.x, h.h0i, fma(GS.y, h.h0r, v[1]));
    if (GEO) {
      const double cr = qS.x * GS.x - qS.y * GS.y, cim = qS.x * GS.y + qS.y * GS.x;
      const double a1 = cr * h.h1r - cim * h.h1i;   // Re(q G H_1)
      e[0] = fma(a1 * ir, dx, e[0]);
      e[1] = fma(a1 * ir, dy, e[1]);
    }
  }
  if (kD) {
    const double f = fma(dx, g.z, dy * g.w) * ir;   // (x - x').n' / rho
    const double wr = GD.x * f, wi = GD.y * f;
    v[2] = fma(wr, h.h1r, fma(-wi, h.h1i, v[2]));
    v[3] = fma(wr, h.h1i, fma(wi, h.h1r, v[3]));
    if (GEO) {
      const double cr = qD.x * GD.x - qD.y * GD.y, cim = qD.x * GD.y + qD.y * GD.x;
      const double a0 = cr * h.h0r - cim * h.h0i;   // Re(q G H_0)
      const double a1 = cr * h.h1r - cim * h.h1i;   // Re(q G H_1)
      const double ux = dx * ir, uy = dy * ir;
      const double b = (k * a0 - 2.0 * a1 * ir) * f;
      e[0] -= fma(b, ux, a1 * ir * g.z);
      e[1] -= fma(b, uy, a1 * ir * g.w);
      e[2] = fma(a1, ux, e[2]);
      e[3] = fma(a1, uy, e[3]);
    }
  }
}

// partial[sp][kk][t]: direct sums of target t over the far sources of panels
// sp, sp + n_fsplit, sp + 2 n_fsplit, ... (interleaved, so that the costly
// panels next to each target's near zone spread over all splits); wave
// gw = sp * n_tb + tb covers targets tb*64 ..
// Per (wave, far panel) a vote: is every active lane at least zt / k from every
// far source of the panel, its nodes (the distance to the panel's mean less its
// node radius bnd.w, with a relative margin for rounding), for the seed fits' thresholds
// zt = 80, 60, 20 in turn?  The first that holds (75%, 9% and 11% of the pairs at
// 4096 panels) gives the panel's pairs that fit with no per-pair vote: the
// coefficient block is addressed once per panel, so its loads stay in scalar
// registers through the panel's loop, and its constant terms are copied into
// vector registers once per panel.  Otherwise (5%) each pair votes as in
// hankel01.  (Panel votes for the z >= 10 and z >= 6 fits as well cost 20 more
// vector registers, one wave a SIMD fewer and 3% of the time; staging the source
// panels in LDS instead of reading them by scalar loads was measured 4% slower.)
template <int KIND>
__global__ __launch_bounds__(256) void k_split_far(const double4* __restrict__ geo,
                                                   const double2* __restrict__ dens, int N,
                                                   const double* __restrict__ nodes, int T,
                                                   const double4* __restrict__ bnd, int NP,
                                                   double g2, double k, int n_tb, int n_fsplit,
                                                   const FarItem* __restrict__ item,
                                                   double2* __restrict__ partial) {
  if (item && !far_off(*item)) return;   // k_split_mid
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + wave;
  const int sp = gw / n_tb;
  const int tb = gw - sp * n_tb;
  if (sp >= n_fsplit) return;
  const int t = tb * kWave + lane;
  const bool valid = t < T;
  const int tt = valid ? t : T - 1;
  const double tx = nodes[2 * (size_t)tt], ty = nodes[2 * (size_t)tt + 1];
  const double4 bt = bnd[tt / kQ];
  const double inv_k = 1.0 / k;
  const double zv = seed::kZV * (1.0 + 1e-12), zu = seed::kZU * (1.0 + 1e-12);
  const double zf = seed::kZF * (1.0 + 1e-12);
  const double2* __restrict__ densD = dens + (kS ? (size_t)N : 0);
  double sr = 0.0, si = 0.0, dr = 0.0, di = 0.0;
  // the pairs of one far panel with one fit block: LEN terms at offset OFF, for z
  // past zt (t = zt / z = (zt / k) / rho)
  auto panel_fit = [&](auto len, auto off, double zt, int j0) {
    constexpr int LEN = decltype(len)::value;
    const double* __restrict__ cf = g_seed_table + opaque_zero();
    const double* __restrict__ fc = cf + decltype(off)::value;
    const D4 c0 = fit_c0(fc);
    const double kt = zt * inv_k;
    for (int b = 0; b < kQ; ++b) {
      const int j = j0 + b;
      const double4 g = geo[j];
      const double dx = tx - g.x, dy = ty - g.y;
      const double rho2 = fma(dx, dx, dy * dy);
      const double ir = rsqrt_refined(rho2);
      const double z = k * (rho2 * ir);
      const H01 h = hankel01_fit_c0<LEN>(z, kt * ir, fc, c0, cf);
      far_accumulate_q<kS, kD>(dens[j], densD[j], g, dx, dy, ir, h, sr, si, dr, di);
    }
  };
  for (int pm = sp; pm < NP; pm += n_fsplit) {
    const double4 bp = bnd[pm];
    const bool far = valid && !panels_near(bt, bp, g2);
    if (far) {
      const int j0 = pm * kQ;
      const double ex = tx - bp.x, ey = ty - bp.y;
      const double e2 = fma(ex, ex, ey * ey);
      const double lo = e2 * rsqrt_refined(e2) - bp.w;
      if (__all(k * lo >= zu)) {
        panel_fit(std::integral_constant<int, seed::kUFARLen>{},
                  std::integral_constant<int, seed::kUFAROff>{}, seed::kZU, j0);
      } else if (__all(k * lo >= zv)) {
        panel_fit(std::integral_constant<int, seed::kVFARLen>{},
                  std::integral_constant<int, seed::kVFAROff>{}, seed::kZV, j0);
      } else if (__all(k * lo >= zf)) {
        panel_fit(std::integral_constant<int, seed::kFARLen>{},
                  std::integral_constant<int, seed::kFAROff>{}, seed::kZF, j0);
      } else {
        for (int b = 0; b < kQ; ++b) {
          const int z0 = opaque_zero();
          const double* __restrict__ cf = g_seed_table + z0;
          const int j = j0 + b;
          const double4 g = geo[j];
          const double dx = tx - g.x, dy = ty - g.y;
          const double rho2 = fma(dx, dx, dy * dy);
          const double ir = rsqrt_refined(rho2);
          const double z = k * (rho2 * ir), iz = ir * inv_k;
          const H01 h = __all(z >= seed::kZV) ? hankel01_vfar(z, iz, cf) : hankel01(z, iz, cf);
          far_accumulate_q<kS, kD>(dens[j], densD[j], g, dx, dy, ir, h, sr, si, dr, di);
        }
      }
    }
  }
  if (valid) {
    int kk = 0;
    if (kS) partial[((size_t)sp * NK + kk++) * T + t] = make_double2(sr, si);
    if (kD) partial[((size_t)sp * NK + kk) * T + t] = make_double2(k * dr, k * di);
  }
}

// parts of the far sums: one with panel expansions (an item), the direct passes' n without or
// where the expansions are off
__device__ __forceinline__ int split_parts(int n, const FarItem* item) {
  return item && !far_off(*item) ? 1 : n;
}

// out[si][kk][t] = (i/4) (near[kk][ci] + sum over far splits of far[sp][kk][t])
__global__ __launch_bounds__(256) void k_split_finalize(int Mc, int T, int nk, int n_fsplit,
                                                        const FarItem* __restrict__ item,
                                                        const double2* __restrict__ nearp,
                                                        const double2* __restrict__ farp,
                                                        double* __restrict__ out) {
  n_fsplit = split_parts(n_fsplit, item);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Mc * nk) return;
  const int kk = e / Mc, ci = e - kk * Mc;
  const int si = ci / T, t = ci - si * T;
  const double2 v0 = nearp[(size_t)kk * Mc + ci];
  double r = v0.x, im = v0.y;
  for (int sp = 0; sp < n_fsplit; ++sp) {
    const double2 v = farp[((size_t)sp * nk + kk) * T + t];
    r += v.x;
    im += v.y;
  }
  const size_t o = ((size_t)si * nk + kk) * T + t;
  out[2 * o] = -0.25 * im;
  out[2 * o + 1] = 0.25 * r;
}

// ---------------------------------------------------------------------------
// Adjoint of the split with respect to the density.  With G_i = conj(g_i) i/4
// (per kind and center) the gradient of L = Re <g, u> with respect to q_j =
// w_j sigma_j is conj(sum_i G_i K_ij), K the pair kernel of whichever rule
// (QBX or direct) the pair takes; the density gradient is then the transposed
// interpolation of w_j conj(...) (PyTorch's convention, A^H g).
// ---------------------------------------------------------------------------

// Gf[kk][t] = sum over the sides of G[kk][si T + t]: the far sums do not depend on
// the side, so their transpose takes the two sides' cotangents together
__global__ __launch_bounds__(256) void k_split_gfar(int T, int nk, int n_sides,
                                                   const double2* __restrict__ G,
                                                   double2* __restrict__ Gf) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= T * nk) return;
  const int kk = e / T, t = e - kk * T;
  const size_t Mc = (size_t)n_sides * T;
  double2 v = G[kk * Mc + t];
  if (n_sides == 2) {
    const double2 w = G[kk * Mc + T + t];
    v = make_double2(v.x + w.x, v.y + w.y);
  }
  Gf[e] = v;
}

// partial[sp][kk][j]: sum over the targets t of far panels in split sp (panels
// sp, sp + n_asplit, ...) of Gf_t K_far(t, j); lanes are 64 consecutive sources,
// targets wave-uniform
// The vote of k_split_far per (wave, target panel); here the targets are the
// panel's nodes, so its node radius bounds them.
// GEO adds the far pairs' gradients for the source's position and normal,
// contracted with its weighted densities q (slots NK and NK + 1 of the split's
// NK + 2): with u = (x - x')/rho, f = u.n' and H_0' = -H_1 (DLMF 10.6.2),
//   d/dx' H_0(k rho) = k H_1 u,
//   d/dx' [k H_1 f] = -k [k H_0 f u + (H_1/rho)(n' - 2 f u)],   d/dn' [k H_1 f] = k H_1 u,
// each summed as Re(q G_t .) over the split's targets.
template <int KIND, bool GEO>
__global__ __launch_bounds__(256) void k_split_far_adj(
    const double4* __restrict__ geo, const double2* __restrict__ dens, int N,
    const double* __restrict__ nodes, int T, const double4* __restrict__ bnd, int NP, double g2,
    double k, const double2* __restrict__ Gf, int n_sb, int n_asplit,
    const FarItem* __restrict__ item, double2* __restrict__ partial) {
  if (item && !far_off(*item)) return;
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  constexpr int NS = NK + (GEO ? 2 : 0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + wave;
  const int sp = gw / n_sb;
  const int sb = gw - sp * n_sb;
  if (sp >= n_asplit) return;
  const int j = sb * kWave + lane;
  const bool valid = j < N;
  const int jj = valid ? j : N - 1;
  const double4 g = geo[jj];
  const double4 bj = bnd[jj / kQ];
  const double inv_k = 1.0 / k;
  const double zv = seed::kZV * (1.0 + 1e-12), zu = seed::kZU * (1.0 + 1e-12);
  const double zf = seed::kZF * (1.0 + 1e-12);
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  double2 qS = make_double2(0.0, 0.0), qD = qS;
  if (GEO) {
    qS = dens[jj];
    qD = dens[(size_t)(NK - 1) * N + jj];
  }
  double e[4] = {0.0, 0.0, 0.0, 0.0};   // GEO: position and normal, without the factor k
  auto add = [&](int t, double dx, double dy, double ir, const H01& h) {
    adj_accumulate<kS, kD, GEO>(Gf[t], Gf[(size_t)(NK - 1) * T + t], qS, qD, g, dx, dy, ir, k, h, v,
                                e);
  };
  for (int mt = sp; mt < NP; mt += n_asplit) {
    const double4 bt = bnd[mt];
    const bool far = valid && !panels_near(bt, bj, g2);
    if (far) {
      // every pair of the active lanes with this target panel at z >= kZV: the
      // distance to the panel's mean less its node radius (the targets are the
      // nodes) bounds |x - x'| from below
      const double ex = g.x - bt.x, ey = g.y - bt.y;
      const double e2 = fma(ex, ex, ey * ey);
      const double lo = e2 * rsqrt_refined(e2) - bt.w;
      // the pairs of this target panel with one fit block (as in k_split_far)
      auto panel_fit = [&](auto len, auto off, double zt) {
        constexpr int LEN = decltype(len)::value;
        const double* __restrict__ cf = g_seed_table + opaque_zero();
        const double* __restrict__ fc = cf + decltype(off)::value;
        const D4 c0 = fit_c0(fc);
        const double kt = zt * inv_k;
        for (int a = 0; a < kQ; ++a) {
          const int t = mt * kQ + a;
          const double dx = nodes[2 * (size_t)t] - g.x, dy = nodes[2 * (size_t)t + 1] - g.y;
          const double rho2 = fma(dx, dx, dy * dy);
          const double ir = rsqrt_refined(rho2);
          const double z = k * (rho2 * ir);
          add(t, dx, dy, ir, hankel01_fit_c0<LEN>(z, kt * ir, fc, c0, cf));
        }
      };
      if (__all(k * lo >= zu)) {
        panel_fit(std::integral_constant<int, seed::kUFARLen>{},
                  std::integral_constant<int, seed::kUFAROff>{}, seed::kZU);
      } else if (__all(k * lo >= zv)) {
        panel_fit(std::integral_constant<int, seed::kVFARLen>{},
                  std::integral_constant<int, seed::kVFAROff>{}, seed::kZV);
      } else if (__all(k * lo >= zf)) {
        panel_fit(std::integral_constant<int, seed::kFARLen>{},
                  std::integral_constant<int, seed::kFAROff>{}, seed::kZF);
      } else {
        for (int a = 0; a < kQ; ++a) {
          const int t = mt * kQ + a;
          const int z0 = opaque_zero();
          const double* __restrict__ cf = g_seed_table + z0;
          const double dx = nodes[2 * (size_t)t] - g.x, dy = nodes[2 * (size_t)t + 1] - g.y;
          const double rho2 = fma(dx, dx, dy * dy);
          const double ir = rsqrt_refined(rho2);
          const double z = k * (rho2 * ir), iz = ir * inv_k;
          add(t, dx, dy, ir,
              __all(z >= seed::kZV) ? hankel01_vfar(z, iz, cf) : hankel01(z, iz, cf));
        }
      }
    }
  }
  if (valid) {
    int kk = 0;
    if (kS) partial[((size_t)sp * NS + kk++) * N + j] = make_double2(v[0], v[1]);
    if (kD) partial[((size_t)sp * NS + kk) * N + j] = make_double2(k * v[2], k * v[3]);
    if (GEO) {
      partial[((size_t)sp * NS + NK) * N + j] = make_double2(k * e[0], k * e[1]);
      partial[((size_t)sp * NS + NK + 1) * N + j] = make_double2(k * e[2], k * e[3]);
    }
  }
}

// grad_density[kk][t] = sum_b V[b][a] w_j conj(acc[kk][j]) (acc in n_acc parts, j = m qs + b, the
// near sources of panel m) + w_t conj(sum_sp partial[sp][kk][t]) (the far source
// at node t = 16 m + a, weight w_t): one thread per node and kind
__global__ __launch_bounds__(256) void k_split_density_grad(
    int T, int N, int qs, int nk, int n_acc, int n_asplit, const FarItem* __restrict__ item,
    const double* __restrict__ tab, const double* __restrict__ wgt, const double* __restrict__ nw,
    const double2* __restrict__ acc, const double2* __restrict__ partial,
    double* __restrict__ grad_density) {
  n_asplit = split_parts(n_asplit, item);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= T * nk) return;
  const TableLayout L = table_layout(qs);
  const int kk = e / T, t = e - kk * T;
  const int m = t / kQ, a = t - m * kQ;
  double gr = 0.0, gi = 0.0;
  for (int b = 0; b < qs; ++b) {
    const size_t j = (size_t)m * qs + b;
    double2 v = make_double2(0.0, 0.0);
    for (int p = 0; p < n_acc; ++p) {
      const double2 x = acc[((size_t)p * nk + kk) * N + j];
      v = make_double2(v.x + x.x, v.y + x.y);
    }
    const double c = tab[L.V + b * kQ + a] * wgt[j];
    gr = fma(c, v.x, gr);
    gi = fma(-c, v.y, gi);      // conj
  }
  double fr = 0.0, fi = 0.0;
  for (int sp = 0; sp < n_asplit; ++sp) {
    const double2 q = partial[((size_t)sp * nk + kk) * T + t];
    fr += q.x;
    fi += q.y;
  }
  const double w = nw[t];
  grad_density[2 * (size_t)e] = fma(w, fr, gr);
  grad_density[2 * (size_t)e + 1] = fma(-w, fi, gi);
}

// ---------------------------------------------------------------------------
// Node gradient of the split.  The loss L = Re sum_i conj(g_i) u_i is a sum over
// pairs, each taken by one rule, so its gradient is the plain adjoint's per-pair
// terms over the near pairs plus the direct rule's over the far ones:
//  * both sides, near pairs (k_near_sources of qbx_near.hip, as the plain adjoint): one
//    evaluation per pair, then the per-center gradients of center_grad_from_sums (target,
//    radius, normal);
//  * far pairs: expansions and their transpose from 96 panels on, with k_split_mid;
//    below, source side k_split_far_adj<KIND, true> over the far sources (the nodes),
//    target side the far target gradients of k_split_far_grad; k_split_nystrom_grad puts both on the
//    nodes (position, normal, the weight's tangent term, the density);
//  * the plain adjoint's k_source_finalize and chain rule (chain_panel) map everything to
//    the nodes and node densities.
// ---------------------------------------------------------------------------

// The far pairs' terms of the node gradient, per node t = 16 m + a (added to
// the first side's center slot t, which the chain rule sums with the other's):
//  * target side: Re(Gf_t . far target gradient) over kinds and far splits, into
//    cg[t][0..1];
//  * source side (the far source at node t), from the far splits' sums of
//    k_split_far_adj<KIND, true>: F_kk (density), the position gradient into
//    cg[t][0..1] and the normal gradient into cg[t][3..4] (the far source's normal
//    is the node's own, as the center's); its weight w = omega_a |X'| enters through
//    g_w = sum_kk Re(F_kk sigma_kk), gtw[t] = g_w omega_a X'/|X'| with X'/|X'| =
//    (-n_y, n_x); gde[kk][t] = w conj(F_kk) joins the node density gradient.
__global__ __launch_bounds__(256) void k_split_nystrom_grad(
    int T, int nk, int n_fsplit, int n_asplit, const FarItem* __restrict__ item,
    const double* __restrict__ density,
    const double4* __restrict__ ngeo, const double* __restrict__ nw,
    const double* __restrict__ w16, const double2* __restrict__ Gf,
    const double2* __restrict__ fpart, const double2* __restrict__ apart,
    double* __restrict__ cg, double* __restrict__ gtw, double2* __restrict__ gde) {
  n_fsplit = split_parts(n_fsplit, item);
  n_asplit = split_parts(n_asplit, item);
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const int ns = nk + 2;
  const double w = nw[t];
  double gx = 0.0, gy = 0.0, gnx = 0.0, gny = 0.0, gw = 0.0;
  for (int kk = 0; kk < nk; ++kk) {
    double xr = 0.0, xi = 0.0, yr = 0.0, yi = 0.0;
    for (int sp = 0; sp < n_fsplit; ++sp) {
      const double2* q = fpart + (((size_t)sp * nk + kk) * T + t) * 2;
      xr += q[0].x;
      xi += q[0].y;
      yr += q[1].x;
      yi += q[1].y;
    }
    const double2 g = Gf[(size_t)kk * T + t];
    gx += g.x * xr - g.y * xi;
    gy += g.x * yr - g.y * yi;
    double fr = 0.0, fi = 0.0;
    for (int sp = 0; sp < n_asplit; ++sp) {
      const double2 v = apart[((size_t)sp * ns + kk) * T + t];
      fr += v.x;
      fi += v.y;
    }
    const double* sg = density + 2 * ((size_t)kk * T + t);
    gw += fr * sg[0] - fi * sg[1];   // Re(F sigma)
    gde[(size_t)kk * T + t] = make_double2(w * fr, -w * fi);
  }
  for (int sp = 0; sp < n_asplit; ++sp) {
    const double2 x = apart[((size_t)sp * ns + nk) * T + t];
    const double2 n = apart[((size_t)sp * ns + nk + 1) * T + t];
    gx += x.x;
    gy += x.y;
    gnx += n.x;
    gny += n.y;
  }
  double* c = cg + (size_t)t * 8;
  c[0] += gx;
  c[1] += gy;
  c[3] += gnx;
  c[4] += gny;
  const double4 g = ngeo[t];
  const double om = w16[t % kQ];
  gtw[2 * (size_t)t] = -gw * om * g.w;
  gtw[2 * (size_t)t + 1] = gw * om * g.z;
}

// ---------------------------------------------------------------------------
// Target derivatives with the split (Section 3.2 for the near sources' local
// expansion, the chain rule for the direct ones).  Near: per center the sums
// F_R = sum q dK/dR and F_theta = sum q dK/dtheta over the near sources
// (grad_source); far: per target
//   S: grad H_0(k rho) = -k H_1 u,   D: grad [k H_1 f] = k [k H_0 f u + (H_1/rho)(n' - 2 f u)],
// u = (x - x')/rho, f = u . n'; the finalize combines them as grad u = (i/4)
// (F_R w^ + (F_theta/R) theta^ + far) and n . grad u with n = -s w^.
// ---------------------------------------------------------------------------

// partial[sp][kk][t][0..1]: the direct gradient (x, y) of target t over the far
// sources of panels sp, sp + n_fsplit, ..., without the factors -k (S), k (D)
template <int KIND>
__global__ __launch_bounds__(256) void k_split_far_grad(
    const double4* __restrict__ geo, const double2* __restrict__ dens, int N,
    const double* __restrict__ nodes, int T, const double4* __restrict__ bnd, int NP, double g2,
    double k, int n_tb, int n_fsplit, const FarItem* __restrict__ item,
    double2* __restrict__ partial) {
  if (item && !far_off(*item)) return;
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + wave;
  const int sp = gw / n_tb;
  const int tb = gw - sp * n_tb;
  if (sp >= n_fsplit) return;
  const int t = tb * kWave + lane;
  const bool valid = t < T;
  const int tt = valid ? t : T - 1;
  const double tx = nodes[2 * (size_t)tt], ty = nodes[2 * (size_t)tt + 1];
  const double4 bt = bnd[tt / kQ];
  const double inv_k = 1.0 / k;
  double S[4] = {0.0, 0.0, 0.0, 0.0}, D[4] = {0.0, 0.0, 0.0, 0.0};
  for (int pm = sp; pm < NP; pm += n_fsplit) {
    const bool far = valid && !panels_near(bt, bnd[pm], g2);
    if (far) {
      const int j0 = pm * kQ;
      for (int b = 0; b < kQ; ++b) {
        const int z0 = opaque_zero();
        const double* __restrict__ cf = g_seed_table + z0;
        const int j = j0 + b;
        const double4 g = geo[j];
        const double dx = tx - g.x, dy = ty - g.y;
        const double rho2 = fma(dx, dx, dy * dy);
        const double ir = rsqrt_refined(rho2);
        const double z = k * (rho2 * ir), iz = ir * inv_k;
        const H01 h = __all(z >= seed::kZV) ? hankel01_vfar(z, iz, cf) : hankel01(z, iz, cf);
        grad_accumulate<kS, kD>(dens[j], dens[(kS && kD ? (size_t)N : 0) + j], g, dx, dy, ir, k, h, S,
                                D);
      }
    }
  }
  if (valid) {
    int kk = 0;
    if (kS) {
      double2* q = partial + (((size_t)sp * NK + kk++) * T + t) * 2;
      q[0] = make_double2(-k * S[0], -k * S[1]);
      q[1] = make_double2(-k * S[2], -k * S[3]);
    }
    if (kD) {
      double2* q = partial + (((size_t)sp * NK + kk) * T + t) * 2;
      q[0] = make_double2(k * D[0], k * D[1]);
      q[1] = make_double2(k * D[2], k * D[3]);
    }
  }
}

// grad[si][kk][t][0..1] and dn[si][kk][t] from the near sums of center ci and the
// far sums of its target
__global__ __launch_bounds__(256) void k_split_finalize_gradient(
    int Mc, int T, int nk, int n_fsplit, const FarItem* __restrict__ item,
    int side, const CenterRec* __restrict__ ctr,
    const double2* __restrict__ nearp, const double2* __restrict__ farp, double* __restrict__ grad,
    double* __restrict__ dn) {
  n_fsplit = split_parts(n_fsplit, item);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Mc * nk) return;
  const int kk = e / Mc, ci = e - kk * Mc;
  const int si = ci / T, t = ci - si * T;
  const double2 F = nearp[((size_t)kk * Mc + ci) * 2], Ft = nearp[((size_t)kk * Mc + ci) * 2 + 1];
  const CenterRec c = ctr[ci];
  const double ir = 1.0 / c.R;
  // F_R w^ + (F_theta / R) theta^, theta^ = (-sin, cos)
  double gxr = fma(F.x, c.ct, -Ft.x * ir * c.st), gxi = fma(F.y, c.ct, -Ft.y * ir * c.st);
  double gyr = fma(F.x, c.st, Ft.x * ir * c.ct), gyi = fma(F.y, c.st, Ft.y * ir * c.ct);
  for (int sp = 0; sp < n_fsplit; ++sp) {
    const double2* q = farp + (((size_t)sp * nk + kk) * T + t) * 2;
    gxr += q[0].x;
    gxi += q[0].y;
    gyr += q[1].x;
    gyi += q[1].y;
  }
  const double s = side != 0 ? (double)side : (si == 0 ? 1.0 : -1.0);
  const size_t o = ((size_t)si * nk + kk) * T + t;
  if (grad) {   // (i/4) z = (-Im z / 4, Re z / 4)
    double* q = grad + 4 * o;
    q[0] = -0.25 * gxi;
    q[1] = 0.25 * gxr;
    q[2] = -0.25 * gyi;
    q[3] = 0.25 * gyr;
  }
  if (dn) {     // n = -s w^
    const double nr = -s * fma(c.ct, gxr, c.st * gyr), ni = -s * fma(c.ct, gxi, c.st * gyi);
    dn[2 * o] = -0.25 * ni;
    dn[2 * o + 1] = 0.25 * nr;
  }
}

// ---------------------------------------------------------------------------
// Far pairs that panel expansions do not take (qbx_far.hip), with those that they do
// already summed per target (fu) or per source (fs): one wave per panel walks the panels
// that are left (few: between gamma panel radii and the expansions' reach), 16 lanes its
// nodes, the four groups of 16 lanes a quarter of the other panel's nodes each.
// Where no expansion reaches many of them (far_off), the direct passes take every far pair.
// MODE 0: values, out[kk][t]; 1: target gradients, out[kk][t][0..1]; 2, 3: the adjoint's
// source side without and with position and normal, out[kk (.. nk + 1)][j].
// ---------------------------------------------------------------------------
template <int KIND, int MODE>
__global__ __launch_bounds__(256) void k_split_mid(FarBlocks B, const double* __restrict__ ro,
                                                   double2* __restrict__ out) {
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int m = b * 4 + wave;
  if (m >= it.P || far_off(it)) return;
  const int T = it.T;
  const int me = m * kQ + (lane & 15), s0 = (lane >> 4) * 4;
  const double4* __restrict__ geo = reinterpret_cast<const double4*>(ro + it.fgeo);
  const double2* __restrict__ dens = reinterpret_cast<const double2*>(ro + it.fdens);
  const double2* __restrict__ Gf = reinterpret_cast<const double2*>(ro + it.fG);
  const double4* __restrict__ bnd = reinterpret_cast<const double4*>(ro + it.bnd);
  const int* __restrict__ count = reinterpret_cast<const int*>(ro + it.mcount);
  const int* __restrict__ list = reinterpret_cast<const int*>(ro + it.mlist) + (size_t)m * kNearCap;
  FarRel R;
  R.r0 = reinterpret_cast<const FarRec*>(ro + it.rec0);
  R.r1 = it.C1 > 0 ? reinterpret_cast<const FarRec*>(ro + it.rec1) : nullptr;
  R.g = it.g;
  R.bnd = bnd;
  R.g2 = it.g2;
  const double k = it.k, inv_k = 1.0 / k;
  const double4 x = geo[me];
  const double2 qS = dens[me], qD = dens[(size_t)(NK - 1) * T + me];
  double u[4] = {0.0, 0.0, 0.0, 0.0}, e[4] = {0.0, 0.0, 0.0, 0.0};
  auto pairs = [&](int pan) {
    if (panels_near(bnd[m], bnd[pan], it.g2)) return;   // a near pair (QBX)
    for (int s = 0; s < 4; ++s) {
      const int z0 = opaque_zero();
      const double* __restrict__ cf = g_seed_table + z0;
      const int j = pan * kQ + s0 + s;
      const double4 y = geo[j];
      // MODE 0, 1: x the target, y the source; 2, 3: x the source, y the target
      const double dx = MODE < 2 ? x.x - y.x : y.x - x.x, dy = MODE < 2 ? x.y - y.y : y.y - x.y;
      const double rho2 = fma(dx, dx, dy * dy);
      const double ir = rsqrt_refined(rho2);
      const H01 h = hankel01(k * (rho2 * ir), ir * inv_k, cf);
      if (MODE == 0)
        far_accumulate_q<kS, kD>(dens[j], dens[(size_t)(NK - 1) * T + j], y, dx, dy, ir, h, u[0],
                                 u[1], u[2], u[3]);
      else if (MODE == 1)
        grad_accumulate<kS, kD>(dens[j], dens[(size_t)(NK - 1) * T + j], y, dx, dy, ir, k, h, u, e);
      else
        adj_accumulate<kS, kD, MODE == 3>(Gf[j], Gf[(size_t)(NK - 1) * T + j], qS, qD, x, dx, dy,
                                          ir, k, h, u, e);
    }
  };
  const int cnt = count[m];
  if (cnt <= kNearCap) {
    for (int i = 0; i < cnt; ++i) pairs(list[i]);
  } else {
    for (int w0 = 0; w0 < it.P; w0 += kWave) {
      const int mp = w0 + lane;
      unsigned long long mask = __ballot(mp < it.P && !far_panels(R, m, mp));
      while (mask) {
        const int pan = w0 + __builtin_ctzll(mask);
        mask &= mask - 1;
        pairs(pan);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    u[i] += __shfl_xor(u[i], 16);
    u[i] += __shfl_xor(u[i], 32);
    if (MODE == 1 || MODE == 3) {
      e[i] += __shfl_xor(e[i], 16);
      e[i] += __shfl_xor(e[i], 32);
    }
  }
  if (lane >= kQ) return;
  const double2* __restrict__ fu = reinterpret_cast<const double2*>(ro + (MODE < 2 ? it.fu : it.fs));
  auto put = [&](size_t o, double r, double i) {
    const double2 f = fu[o];
    out[o] = make_double2(f.x + r, f.y + i);
  };
  if (MODE == 1) {
    if (kS) {
      put(2 * (size_t)me, -k * u[0], -k * u[1]);
      put(2 * (size_t)me + 1, -k * u[2], -k * u[3]);
    }
    if (kD) {
      put(2 * ((size_t)(NK - 1) * T + me), k * e[0], k * e[1]);
      put(2 * ((size_t)(NK - 1) * T + me) + 1, k * e[2], k * e[3]);
    }
  } else {
    if (kS) put(me, u[0], u[1]);
    if (kD) put((size_t)(NK - 1) * T + me, k * u[2], k * u[3]);
    if (MODE == 3) {
      put((size_t)NK * T + me, k * e[0], k * e[1]);
      put((size_t)(NK + 1) * T + me, k * e[2], k * e[3]);
    }
  }
}

template <int MODE>
static hipError_t launch_mid(const SplitCall& c, double2* out, hipStream_t s) {
  const dim3 grid((unsigned)((c.d.P + 3) / 4)), block(256);
  const FarBlocks B{c.dev, nullptr, 1};
  switch (c.d.kind) {
    case 1: hipLaunchKernelGGL((k_split_mid<1, MODE>), grid, block, 0, s, B, c.ws, out); break;
    case 2: hipLaunchKernelGGL((k_split_mid<2, MODE>), grid, block, 0, s, B, c.ws, out); break;
    default: hipLaunchKernelGGL((k_split_mid<3, MODE>), grid, block, 0, s, B, c.ws, out); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_nystrom_sources(const Dims& d, const double* nodes, const double* density,
                                  const double* tables, double4* bnd, NystromSources ns,
                                  hipStream_t s) {
  const TableLayout L = table_layout(d.qs);
  hipLaunchKernelGGL(k_nystrom_sources, dim3((d.T + 255) / 256), dim3(256), 0, s, d.T, d.nk,
                     nodes, density, tables + L.Dn, tables + L.w16, bnd, ns.geo, ns.dens, ns.w);
  return hipGetLastError();
}

hipError_t launch_near_lists(const Dims& d, const double4* bnd, double g2, int* count, int* list,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_near_lists, dim3((unsigned)((d.P + 3) / 4)), dim3(256), 0, s, d.P, bnd,
                     g2, count, list);
  return hipGetLastError();
}

hipError_t launch_split_gfar(const Dims& d, const double2* G, double2* Gf, hipStream_t s) {
  const int nt = d.T * d.nk;
  hipLaunchKernelGGL(k_split_gfar, dim3((nt + 255) / 256), dim3(256), 0, s, d.T, d.nk, d.n_sides,
                     G, Gf);
  return hipGetLastError();
}

// one wave per 64 points and source (target) split
static dim3 far_grid(const Dims& d, int splits) {
  const long waves = (long)((d.T + kWave - 1) / kWave) * splits;
  return dim3((unsigned)((waves + 3) / 4));
}

hipError_t launch_split_far(const SplitCall& c, double2* out, hipStream_t s) {
  if (c.far) {
    const hipError_t e = launch_mid<0>(c, out, s);
    if (e != hipSuccess) return e;
  }
  const Dims& d = c.d;
  const int n_tb = (d.T + kWave - 1) / kWave;
  const dim3 grid = far_grid(d, d.n_fsplit), block(256);
#define QBX_FAR_ARGS \
  c.ns.geo, c.ns.dens, d.T, c.nodes, d.T, c.bnd, d.P, c.g2, d.k, n_tb, d.n_fsplit, c.item(), out
  switch (d.kind) {
    case 1: hipLaunchKernelGGL((k_split_far<1>), grid, block, 0, s, QBX_FAR_ARGS); break;
    case 2: hipLaunchKernelGGL((k_split_far<2>), grid, block, 0, s, QBX_FAR_ARGS); break;
    default: hipLaunchKernelGGL((k_split_far<3>), grid, block, 0, s, QBX_FAR_ARGS); break;
  }
  return hipGetLastError();
}

hipError_t launch_split_far_grad(const SplitCall& c, double2* out, hipStream_t s) {
  if (c.far) {
    const hipError_t e = launch_mid<1>(c, out, s);
    if (e != hipSuccess) return e;
  }
  const Dims& d = c.d;
  const int n_tb = (d.T + kWave - 1) / kWave;
  const dim3 grid = far_grid(d, d.n_fsplit), block(256);
  switch (d.kind) {
    case 1: hipLaunchKernelGGL((k_split_far_grad<1>), grid, block, 0, s, QBX_FAR_ARGS); break;
    case 2: hipLaunchKernelGGL((k_split_far_grad<2>), grid, block, 0, s, QBX_FAR_ARGS); break;
    default: hipLaunchKernelGGL((k_split_far_grad<3>), grid, block, 0, s, QBX_FAR_ARGS); break;
  }
#undef QBX_FAR_ARGS
  return hipGetLastError();
}

hipError_t launch_split_far_adj(const SplitCall& c, bool geo, const double2* Gf, double2* out,
                                hipStream_t s) {
  if (c.far) {
    const hipError_t e = geo ? launch_mid<3>(c, out, s) : launch_mid<2>(c, out, s);
    if (e != hipSuccess) return e;
  }
  const Dims& d = c.d;
  const int n_sb = (d.T + kWave - 1) / kWave;
  const dim3 grid = far_grid(d, d.n_asplit), block(256);
#define QBX_FADJ(KD, GEO)                                                                       \
  hipLaunchKernelGGL((k_split_far_adj<KD, GEO>), grid, block, 0, s, c.ns.geo, c.ns.dens, d.T,    \
                     c.nodes, d.T, c.bnd, d.P, c.g2, d.k, Gf, n_sb, d.n_asplit, c.item(),   \
                     out)
  switch (d.kind + (geo ? 4 : 0)) {
    case 1: QBX_FADJ(1, false); break;
    case 2: QBX_FADJ(2, false); break;
    case 3: QBX_FADJ(3, false); break;
    case 5: QBX_FADJ(1, true); break;
    case 6: QBX_FADJ(2, true); break;
    default: QBX_FADJ(3, true); break;
  }
#undef QBX_FADJ
  return hipGetLastError();
}

hipError_t launch_split_finalize(const SplitCall& c, const double2* nearp, const double2* farp,
                                 double* out, hipStream_t s) {
  const Dims& d = c.d;
  const int n = d.Mc * d.nk;
  hipLaunchKernelGGL(k_split_finalize, dim3((n + 255) / 256), dim3(256), 0, s, d.Mc, d.T, d.nk,
                     d.n_fsplit, c.item(), nearp, farp, out);
  return hipGetLastError();
}

hipError_t launch_split_finalize_gradient(const SplitCall& c, const CenterRec* ctr,
                                          const double2* nearp, const double2* farp, double* grad,
                                          double* dn, hipStream_t s) {
  const Dims& d = c.d;
  const int n = d.Mc * d.nk;
  hipLaunchKernelGGL(k_split_finalize_gradient, dim3((n + 255) / 256), dim3(256), 0, s, d.Mc, d.T,
                     d.nk, d.n_fsplit, c.item(), d.side, ctr, nearp, farp, grad, dn);
  return hipGetLastError();
}

hipError_t launch_split_density_grad(const SplitCall& c, const double* tables, const double* wgt,
                                     int n_acc, const double2* acc, const double2* partial,
                                     double* grad_density, hipStream_t s) {
  const Dims& d = c.d;
  const int nt = d.T * d.nk;
  hipLaunchKernelGGL(k_split_density_grad, dim3((nt + 255) / 256), dim3(256), 0, s, d.T, d.N, d.qs,
                     d.nk, n_acc, d.n_asplit, c.item(), tables, wgt, c.ns.w, acc, partial,
                     grad_density);
  return hipGetLastError();
}

hipError_t launch_split_nystrom_grad(const SplitCall& c, const double* density,
                                     const double* tables, const double2* Gf,
                                     const double2* fpart, const double2* apart, double* cg,
                                     double* gtw, double2* gde, hipStream_t s) {
  const Dims& d = c.d;
  const TableLayout L = table_layout(d.qs);
  hipLaunchKernelGGL(k_split_nystrom_grad, dim3((d.T + 255) / 256), dim3(256), 0, s, d.T, d.nk,
                     d.n_fsplit, d.n_asplit, c.item(), density, c.ns.geo, c.ns.w,
                     tables + L.w16, Gf, fpart, apart, cg, gtw, gde);
  return hipGetLastError();
}

}  // namespace qbx
