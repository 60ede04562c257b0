// Stored local expansions (Section 5: one local expansion serving several nearby
// targets).  The coefficients a_l, l = -p..p, of every center (Section 2, eq.
// graf-coefficient; Section 3.2, eq. graf-coefficient-dlp) are formed once and
// kept; any target inside a center's disk is then evaluated from them by Section
// 3.3 step 4(c), with its own distance and angle from the center.
//
//  * A pair (center c, source x') with v = x' - c, rho = |v| and E = e^{-i arg v} has the
//    factors f_m = H_m(k rho) E^m and f_{-m} = (-1)^m H_m(k rho) conj(E)^m.  The single layer
//    adds q f_l to a_l, q = w sigma; the double layer's ladder d/dn' f_l =
//    (k/2)(conj(nu) f_{l-1} - nu f_{l+1}), nu = n_x + i n_y, adds the f_m to its two
//    neighbours with the weights w mu conj(nu) and w mu nu (coef_pair, k/2 in
//    k_coef_finalize).  With D a wave takes one sign of the orders: f_{-m} follows f_m's
//    recurrences with the signs of H_1, of 1/z and of E's imaginary part turned, so one code has
//    both, the sums of both kinds stay in registers up to p = 24, and a pair's H and E serve both
//    kinds.  S alone has room for both signs in one wave, which share f_m's four products.
//  * k_coef: lanes are 64 centers, the sources of a source split are wave-uniform (scalar
//    loads): every pair, where panel expansions do not apply (far_applies_coef).
//  * k_coef_near: the sources of near panels only, where panel expansions take the far ones
//    (qbx_far.hip: the coefficients are the local expansions that those end in).  Near is what
//    keeps each order right by itself (qbx_coef_table.h), which is wider than for potentials.
//  * k_evaluate_expansions: one thread per target,
//    u = (i/4) sum_l a_l J_l(k|x - c|) e^{i l arg(x - c)} with J_l by Miller's
//    recurrence (J_{-l} = (-1)^l J_l).
//  * k_assign_centers: per target, the nearest center whose disk holds it (ties to the
//    lower index), or -1.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "../../include/qbx.h"
#include "qbx_internal.h"
#include "qbx_near.h"
#include "qbx_panel.h"
#include "qbx_special.h"

namespace qbx {

// sums of one sign of the orders: S[l] = a^S_{sg l}, D[l] = (2/k) a^D_{sg l}, 0 <= l <= P (the
// order-0 sums are in parts: S's in the positive sign's, D's in both); S alone: M[l] = a^S_{-l}
template <int P, int KIND>
struct CoefSums {
  double sr[KIND & 1 ? P + 1 : 1], si[KIND & 1 ? P + 1 : 1];
  double dr[KIND & 2 ? P + 1 : 1], di[KIND & 2 ? P + 1 : 1];
  double mr[KIND == 1 ? P + 1 : 1], mi[KIND == 1 ? P + 1 : 1];
};
// waves that share a center's orders
constexpr int coef_halves(int kind) { return kind == 1 ? 1 : 2; }

// adds one pair; q the weighted densities (S, D), sg the sign of the orders (S alone: 1)
template <int P, int KIND>
__device__ __forceinline__ void coef_pair(const double4 g, const double2 qS, const double2 w,
                                          double cx, double cy, double k, double inv_k, double sg,
                                          CoefSums<P, KIND>& A) {
  constexpr bool kS = (KIND & 1) != 0, kD = (KIND & 2) != 0;
  constexpr int M = kD ? P + 1 : P;
  const int z0 = opaque_zero();
  const double* __restrict__ cf = g_seed_table + z0;
  // D: f_m's weight in order m + 1 and, negative, in order m - 1: w conj(nu) and w nu, for the
  // negative orders -w nu and -w conj(nu)
  const double ny = sg * g.w, wx = sg * w.x, wy = sg * w.y;
  const double ur = fma(wx, g.z, wy * ny), ui = fma(wy, g.z, -wx * ny);
  const double lr = fma(wx, g.z, -wy * ny), li = fma(wy, g.z, wx * ny);
  const double vx = g.x - cx, vy = g.y - cy;
  const double rho2 = fma(vx, vx, vy * vy);
  const double ir = rsqrt_refined(rho2);
  const double z = k * (rho2 * ir), iz = ir * inv_k;
  const H01 h = hankel01(z, iz, cf);
  const double e1r = vx * ir, e1i = -sg * (vy * ir);
  const double tz = 2.0 * sg * iz;
  double hpr = h.h0r, hpi = h.h0i, hr = sg * h.h1r, hi = sg * h.h1i;   // H_{m-1}, H_m
  double er = e1r, ei = e1i;                                         // E^m
  if (kS && sg > 0.0) {
    A.sr[0] = fma(qS.x, hpr, fma(-qS.y, hpi, A.sr[0]));
    A.si[0] = fma(qS.x, hpi, fma(qS.y, hpr, A.si[0]));
  }
  if (kD && P >= 1) {
    A.dr[1] = fma(ur, hpr, fma(-ui, hpi, A.dr[1]));
    A.di[1] = fma(ur, hpi, fma(ui, hpr, A.di[1]));
  }
#pragma unroll
  for (int m = 1; m <= M; ++m) {
    const double rr = hr * er, ii = hi * ei, ri = hr * ei, im = hi * er;
    const double fr = rr - ii, fi = ri + im;
    if (KIND == 1) {   // f_{-m} = (-1)^m H_m conj(E)^m
      const double qx = (m & 1) ? -qS.x : qS.x, qy = (m & 1) ? -qS.y : qS.y;
      const double gr = rr + ii, gi = im - ri;
      A.mr[m] = fma(qx, gr, fma(-qy, gi, A.mr[m]));
      A.mi[m] = fma(qx, gi, fma(qy, gr, A.mi[m]));
    }
    if (kS && m <= P) {
      A.sr[m] = fma(qS.x, fr, fma(-qS.y, fi, A.sr[m]));
      A.si[m] = fma(qS.x, fi, fma(qS.y, fr, A.si[m]));
    }
    if (kD) {
      A.dr[m - 1] = fma(-lr, fr, fma(li, fi, A.dr[m - 1]));
      A.di[m - 1] = fma(-lr, fi, fma(-li, fr, A.di[m - 1]));
      if (m + 1 <= P) {
        A.dr[m + 1] = fma(ur, fr, fma(-ui, fi, A.dr[m + 1]));
        A.di[m + 1] = fma(ur, fi, fma(ui, fr, A.di[m + 1]));
      }
    }
    if (m < M) {
      // H_{m+1} = (2m/z) H_m - H_{m-1};  E^{m+1} = E^m E
      const double t = m * tz;
      const double nr = fma(t, hr, -hpr), ni = fma(t, hi, -hpi);
      hpr = hr;
      hpi = hi;
      hr = nr;
      hi = ni;
      const double tr = fma(er, e1r, -ei * e1i);
      ei = fma(er, e1i, ei * e1r);
      er = tr;
    }
  }
}

template <int P, int KIND>
__device__ __forceinline__ void coef_zero(CoefSums<P, KIND>& A) {
#pragma unroll
  for (int l = 0; l <= P; ++l) {
    if (KIND & 1) A.sr[l] = A.si[l] = 0.0;
    if (KIND & 2) A.dr[l] = A.di[l] = 0.0;
    if (KIND == 1) A.mr[l] = A.mi[l] = 0.0;
  }
}

// partial[sp][half][kind][l][ci]
template <int P, int KIND>
__device__ __forceinline__ void coef_store(const CoefSums<P, KIND>& A, int sp, int half, int ci,
                                           int Mc, double2* __restrict__ partial) {
  constexpr int NK = KIND == 3 ? 2 : 1;
  double2* o = partial + ((size_t)(sp * 2 + half) * NK * (P + 1)) * Mc + ci;
#pragma unroll
  for (int l = 0; l <= P; ++l) {
    if (KIND & 1) o[(size_t)l * Mc] = make_double2(A.sr[l], A.si[l]);
    if (KIND == 1) o[(size_t)(P + 1 + l) * Mc] = make_double2(A.mr[l], A.mi[l]);
    if (KIND & 2) o[(size_t)((NK - 1) * (P + 1) + l) * Mc] = make_double2(A.dr[l], A.di[l]);
  }
}

// the sums over the sources of split sp; q: [n kinds][N] weighted densities
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_coef(const double4* __restrict__ geo,
                                              const double2* __restrict__ q, int N,
                                              const CenterRec* __restrict__ ctr, int Mc,
                                              int n_cb, int n_sp, int src_per_split, double k,
                                              double2* __restrict__ partial) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + wave;
  constexpr int kH = coef_halves(KIND);
  const int half = gw % kH;
  const int sp = gw / kH / n_cb;
  const int cb = gw / kH - sp * n_cb;
  const int ci = cb * kWave + lane;
  if (sp >= n_sp) return;   // past the last split (whole waves); an empty split writes zeros
  const int j0 = sp * src_per_split;
  const int j1 = min(N, j0 + src_per_split);
  const bool valid = ci < Mc;
  const CenterRec c = ctr[valid ? ci : Mc - 1];
  const double inv_k = 1.0 / k, sg = half ? -1.0 : 1.0;
  const double2* __restrict__ qD = q + (KIND == 3 ? (size_t)N : 0);
  CoefSums<P, KIND> A;
  coef_zero<P, KIND>(A);
  for (int j = j0; j < j1; ++j)
    coef_pair<P, KIND>(geo[j], q[j], qD[j], c.cx, c.cy, k, inv_k, sg, A);
  if (valid) coef_store<P, KIND>(A, sp, half, ci, Mc, partial);
}

// The sums over the sources of panels near the center's; a wave has the 16 centers of one panel
// and side, four lanes each, and of each near panel the sources 4 sp + (0..3) + 4 n_sp i (whole
// panels dealt to the splits left some with twice the work).  Bound by FP64 issue and its
// latency at two waves a SIMD: 213 VGPRs at p = 12, S + D.  256 panels, k = 20, both sides, all
// kernels: 1.75 ms with the 73 panels of p = 12 near, 4.4 over every pair (k_coef), 8.0 as three
// passes over every pair (one per weight).
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_coef_near(FarBlocks B, const double* __restrict__ ro,
                                                   int n_sp, double2* __restrict__ partial) {
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = b * 4 + wave;
  constexpr int kH = coef_halves(KIND);
  const int half = gw % kH;
  const int sp = gw / kH % n_sp, row = gw / kH / n_sp;
  const int si = row / it.P, m = row - si * it.P;
  if (si >= it.n_sides) return;
  const int ci = si * it.T + m * kQ + (lane & 15);
  const CenterRec c = reinterpret_cast<const CenterRec*>(ro + it.ctr)[ci];
  const double4* __restrict__ geo = reinterpret_cast<const double4*>(ro + it.geo);
  const double2* __restrict__ q = reinterpret_cast<const double2*>(ro + it.dens);
  const double2* __restrict__ qD = q + (KIND == 3 ? (size_t)it.N : 0);
  const double k = it.k, inv_k = 1.0 / k, sg = half ? -1.0 : 1.0;
  const int qs = it.qs;
  CoefSums<P, KIND> A;
  coef_zero<P, KIND>(A);
  for_near_runs(m, near_rel(it, ro), it.P, near_lists(it, ro), lane, [&](int pan, int n) {
    for (int s = 4 * sp + (lane >> 4); s < n * qs; s += 4 * n_sp) {
      const int j = pan * qs + s;
      coef_pair<P, KIND>(geo[j], q[j], qD[j], c.cx, c.cy, k, inv_k, sg, A);
    }
  });
#pragma unroll
  for (int l = 0; l <= P; ++l)
#pragma unroll
    for (int off = 16; off <= 32; off *= 2) {
      if (KIND & 1) {
        A.sr[l] += __shfl_xor(A.sr[l], off);
        A.si[l] += __shfl_xor(A.si[l], off);
      }
      if (KIND & 2) {
        A.dr[l] += __shfl_xor(A.dr[l], off);
        A.di[l] += __shfl_xor(A.di[l], off);
      }
      if (KIND == 1) {
        A.mr[l] += __shfl_xor(A.mr[l], off);
        A.mi[l] += __shfl_xor(A.mi[l], off);
      }
    }
  if (lane < kQ) coef_store<P, KIND>(A, sp, half, ci, it.Mc, partial);
}

// coef[kk][ci][l + p] from the split sums, added to the far sums that coef holds already where
// the call has an item and its expansions are on.
// A block has 16 centers of one kind: read by runs of centers, written by runs of orders.
__global__ __launch_bounds__(256) void k_coef_finalize(int Mc, int p, int kind, int n_sp,
                                                       double k, const FarItem* item,
                                                       const double2* __restrict__ partial,
                                                       double2* __restrict__ coef) {
  const bool far = item && !far_off(*item);
  __shared__ double2 a[(2 * kPMax + 1) * 16];
  const int nk = kind == 3 ? 2 : 1, L = 2 * p + 1;
  const int kk = blockIdx.y, c0 = blockIdx.x * 16;
  const double f = (kind & 2) && kk == nk - 1 ? 0.5 * k : 1.0;
  for (int t = threadIdx.x; t < L * 16; t += blockDim.x) {
    const int l = t / 16 - p, ci = c0 + t % 16;
    double r = 0.0, im = 0.0;
    if (ci < Mc)
      for (int sp = 0; sp < n_sp; ++sp)
        for (int half = l < 0 ? 1 : 0; half <= (l <= 0 ? 1 : 0); ++half) {
          const double2 v =
              partial[(((size_t)(sp * 2 + half) * nk + kk) * (p + 1) + abs(l)) * Mc + ci];
          r += v.x;
          im += v.y;
        }
    a[t % 16 * L + t / 16] = make_double2(f * r, f * im);
  }
  __syncthreads();
  double2* o = coef + ((size_t)kk * Mc + c0) * L;
  const int n = min(16, Mc - c0) * L;
  for (int t = threadIdx.x; t < n; t += blockDim.x) {
    const double2 v = a[t], w = far ? o[t] : make_double2(0.0, 0.0);
    o[t] = make_double2(w.x + v.x, w.y + v.y);
  }
}

// ctr_xy [Mc][2], ctr_r [Mc] from the center records (either may be NULL)
__global__ __launch_bounds__(256) void k_center_out(int Mc, const CenterRec* __restrict__ ctr,
                                                    double* __restrict__ xy,
                                                    double* __restrict__ rad) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Mc) return;
  const CenterRec c = ctr[i];
  if (xy) {
    xy[2 * (size_t)i] = c.cx;
    xy[2 * (size_t)i + 1] = c.cy;
  }
  if (rad) rad[i] = c.R;
}

// out[kk][t] = (i/4) sum_{l=-p..p} a_l J_l(k R) e^{i l theta}, R e^{i theta} = x_t - c;
// a center index outside [0, Mc) gives NaN
__global__ __launch_bounds__(256) void k_evaluate_expansions(
    int Mc, const double* __restrict__ ctr_xy, const double2* __restrict__ coef, double k,
    int p, int nk, int n_t, const double* __restrict__ tgt, const int32_t* __restrict__ idx,
    double2* __restrict__ out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_t) return;
  const int ci = idx[t];
  if (ci < 0 || ci >= Mc) {
    for (int kk = 0; kk < nk; ++kk) out[(size_t)kk * n_t + t] = make_double2(NAN, NAN);
    return;
  }
  const int L = 2 * p + 1;
  const double dx = tgt[2 * (size_t)t] - ctr_xy[2 * (size_t)ci];
  const double dy = tgt[2 * (size_t)t + 1] - ctr_xy[2 * (size_t)ci + 1];
  const double R = sqrt(dx * dx + dy * dy);
  const double c1 = R > 0.0 ? dx / R : 1.0, s1 = R > 0.0 ? dy / R : 0.0;
  double J[kPMax + 1];
  bessel_j_miller(k * R, p, J);
  for (int kk = 0; kk < nk; ++kk) {
    const double2* a = coef + ((size_t)kk * Mc + ci) * L;
    const double2 a0 = a[p];
    double ur = a0.x * J[0], ui = a0.y * J[0];
    double er = 1.0, ei = 0.0;   // e^{i l theta}
    for (int l = 1; l <= p; ++l) {
      const double tr = er * c1 - ei * s1;
      ei = er * s1 + ei * c1;
      er = tr;
      const double2 ap = a[p + l], am = a[p - l];
      const double jl = J[l], jm = (l & 1) ? -J[l] : J[l];   // J_{-l} = (-1)^l J_l
      // a_l J_l e^{il theta} + a_{-l} J_{-l} e^{-il theta}
      ur += jl * (ap.x * er - ap.y * ei) + jm * (am.x * er + am.y * ei);
      ui += jl * (ap.x * ei + ap.y * er) + jm * (am.y * er - am.x * ei);
    }
    out[(size_t)kk * n_t + t] = make_double2(-0.25 * ui, 0.25 * ur);   // (i/4) u
  }
}

// the nearest center with |x_t - c| <= slack R_c, ties to the lower index; -1 if none.
// Every product and sum is rounded on its own (no contraction), so any IEEE double
// evaluation of the same formula takes the same decisions.
// A wave has NT targets: each center that it reads serves all of them.  Bound by those reads
// (24 bytes a center and wave): 20001 targets and 8192 centers take 77 us, 182 us with one
// target a wave.
template <int NT>
__global__ __launch_bounds__(256) void k_assign_centers(int Mc, const double* __restrict__ ctr_xy,
                                                        const double* __restrict__ ctr_r,
                                                        double slack, int n_t,
                                                        const double* __restrict__ tgt,
                                                        int32_t* __restrict__ idx) {
#pragma clang fp contract(off)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int t0 = (blockIdx.x * 4 + wave) * NT;
  if (t0 >= n_t) return;
  double tx[NT], ty[NT], best[NT];
  int bi[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const size_t t = min(t0 + u, n_t - 1);
    tx[u] = tgt[2 * t];
    ty[u] = tgt[2 * t + 1];
    best[u] = INFINITY;
    bi[u] = -1;
  }
  for (int i = lane; i < Mc; i += kWave) {
    const double cx = ctr_xy[2 * (size_t)i], cy = ctr_xy[2 * (size_t)i + 1];
    const double rr = slack * ctr_r[i];
    const double r2 = rr * rr;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const double dx = tx[u] - cx, dy = ty[u] - cy;
      const double d2 = dx * dx + dy * dy;
      if (d2 <= r2 && d2 < best[u]) {   // lanes visit their centers in increasing order
        best[u] = d2;
        bi[u] = i;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    for (int off = 32; off > 0; off >>= 1) {
      const double ob = __shfl_xor(best[u], off);
      const int oi = __shfl_xor(bi[u], off);
      if (ob < best[u] || (ob == best[u] && oi >= 0 && (bi[u] < 0 || oi < bi[u]))) {
        best[u] = ob;
        bi[u] = oi;
      }
    }
    if (lane == 0 && t0 + u < n_t) idx[t0 + u] = bi[u];
  }
}

namespace {

template <int P, int KIND>
hipError_t launch_coef_k(const Dims& d, bool far, const FarItem* dev, const double* ws,
                         const double4* geo, const double2* q, const CenterRec* ctr, int n_sp,
                         double2* partial, hipStream_t s) {
  if (far) {
    const long waves = (long)coef_halves(KIND) * d.P * d.n_sides * n_sp;
    hipLaunchKernelGGL((k_coef_near<P, KIND>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s,
                       FarBlocks{dev, nullptr, 1}, ws, n_sp, partial);
  } else {
    const int n_cb = (d.Mc + kWave - 1) / kWave;
    const long waves = (long)coef_halves(KIND) * n_cb * n_sp;
    hipLaunchKernelGGL((k_coef<P, KIND>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, geo,
                       q, d.N, ctr, d.Mc, n_cb, n_sp, (d.N + n_sp - 1) / n_sp, d.k, partial);
  }
  return hipGetLastError();
}

template <int P>
hipError_t launch_coef_p(const Dims& d, bool far, const FarItem* dev, const double* ws,
                         const double4* geo, const double2* q, const CenterRec* ctr, int n_sp,
                         double2* partial, hipStream_t s) {
  if (d.kind == 1) return launch_coef_k<P, 1>(d, far, dev, ws, geo, q, ctr, n_sp, partial, s);
  if (d.kind == 2) return launch_coef_k<P, 2>(d, far, dev, ws, geo, q, ctr, n_sp, partial, s);
  return launch_coef_k<P, 3>(d, far, dev, ws, geo, q, ctr, n_sp, partial, s);
}

hipError_t launch_coef(const Dims& d, bool far, const FarItem* dev, const double* ws,
                       const double4* geo, const double2* q, const CenterRec* ctr, int n_sp,
                       double2* partial, hipStream_t s) {
  switch (d.p) {
#define QBX_CASE(PP) \
  case PP:           \
    return launch_coef_p<PP>(d, far, dev, ws, geo, q, ctr, n_sp, partial, s);
    QBX_CASE(0) QBX_CASE(1) QBX_CASE(2) QBX_CASE(3) QBX_CASE(4) QBX_CASE(5) QBX_CASE(6)
    QBX_CASE(7) QBX_CASE(8) QBX_CASE(9) QBX_CASE(10) QBX_CASE(11) QBX_CASE(12) QBX_CASE(13)
    QBX_CASE(14) QBX_CASE(15) QBX_CASE(16) QBX_CASE(17) QBX_CASE(18) QBX_CASE(19) QBX_CASE(20)
    QBX_CASE(21) QBX_CASE(22) QBX_CASE(23) QBX_CASE(24)
#undef QBX_CASE
    default:
      return hipErrorInvalidValue;
  }
}

// splits of the coefficient sums: enough waves (64 centers each, or far a panel and side; with
// D one per sign) to fill the device about four times, at most 8 (the split sums take
// n_sp x 2 x (p + 1) x Mc x 16 bytes per kind)
int coef_splits(const Dims& d, bool far) {
  const int n_cb = coef_halves(d.kind) * (far ? d.P * d.n_sides : (d.Mc + kWave - 1) / kWave);
  int n_sp = std::min(8, (4096 + n_cb - 1) / n_cb);
  const int most = far ? (d.qs + 3) / 4 : (d.N + kWave - 1) / kWave;
  return std::max(1, std::min(n_sp, most));
}

struct ExpLayout {
  Layout base;          // tables .. partial of make_forward_layout (partial unused)
  size_t part, total;
};

ExpLayout make_expansion_layout(const Dims& d) {
  ExpLayout E;
  E.base = make_forward_layout(d, far_coef_size(d));
  // at any r and k, whichever way the sums are formed then
  const size_t n_sp = std::max(coef_splits(d, false), coef_splits(d, true));
  E.part = E.base.total;
  E.total = align256(E.part + sizeof(double2) * n_sp * 2 * d.nk * (d.p + 1) * d.Mc);
  return E;
}

template <typename T>
T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

}  // namespace
}  // namespace qbx

using namespace qbx;

extern "C" {

size_t qbx_expansion_workspace_bytes(int n_panels, int q, int p, int oversample, int side,
                                     int kind) {
  Dims d;
  if (!make_dims(n_panels, q, p, oversample, side, kind, 1.0, 0.5, &d)) return 0;
  return make_expansion_layout(d).total;
}

int qbx_expansion_coefficients(const qbx_geometry* g, const double* density, double k, int p,
                               double r, int oversample, int side, int kind, double* coef,
                               double* ctr_xy, double* ctr_r, void* ws, size_t ws_bytes,
                               hipStream_t stream) {
  Dims d;
  int rc = validate(g, p, k, r, oversample, side, kind, &d);
  if (rc) return rc;
  if (!density) return fail(QBX_EINVAL, "density is NULL");
  if (!coef) return fail(QBX_EINVAL, "coef is NULL");
  if (!ws) return fail(QBX_EINVAL, "workspace is NULL");
  const ExpLayout E = make_expansion_layout(d);
  if (ws_bytes < E.total)
    return fail(QBX_EWORKSPACE, "workspace of %zu bytes, %zu needed", ws_bytes, E.total);
  const Layout& L = E.base;
  const bool far = far_applies_coef(d);
  FarItem it{};
  if (far) {
    it = far_item_of(d, L, false, true, false);
    it.coef = d.p;
  }
  FarItem* dev = far ? at<FarItem>(ws, L.far) : nullptr;
  hipError_t e = launch_tables(d, at<double>(ws, L.tables), stream);
  if (e != hipSuccess) return device_fail(e, "tables kernel");
  e = launch_upsample(d, g->nodes, density, at<double>(ws, L.tables), at<double4>(ws, L.geo),
                      at<double2>(ws, L.dens), at<double>(ws, L.wgt), at<double>(ws, L.h),
                      at<CenterRec>(ws, L.ctr), at<double>(ws, L.jtab), stream,
                      far ? &it : nullptr, dev);
  if (e != hipSuccess) return device_fail(e, "upsample kernel");
  if (far) {
    e = far_fields(far_single(it, dev), g->nodes, static_cast<double*>(ws), true, false, 3, false,
                   false, true, stream, reinterpret_cast<double2*>(coef));
    if (e != hipSuccess) return device_fail(e, "panel expansion kernels");
  }
  const int n_sp = coef_splits(d, far);
  const CenterRec* ctr = at<CenterRec>(ws, L.ctr);
  e = launch_coef(d, far, dev, static_cast<double*>(ws), at<double4>(ws, L.geo),
                  at<double2>(ws, L.dens), ctr, n_sp, at<double2>(ws, E.part), stream);
  if (e != hipSuccess) return device_fail(e, "coefficient kernel");
  hipLaunchKernelGGL(k_coef_finalize, dim3((d.Mc + 15) / 16, d.nk), dim3(256), 0, stream, d.Mc,
                     d.p, d.kind, n_sp, d.k, dev,
                     at<double2>(ws, E.part),
                     reinterpret_cast<double2*>(coef));
  if (ctr_xy || ctr_r)
    hipLaunchKernelGGL(k_center_out, dim3((d.Mc + 255) / 256), dim3(256), 0, stream, d.Mc, ctr,
                       ctr_xy, ctr_r);
  e = hipGetLastError();
  return e == hipSuccess ? QBX_OK : device_fail(e, "coefficient finalize kernels");
}

int qbx_evaluate_expansions(int n_ctr, const double* ctr_xy, const double* coef, double k,
                            int p, int kind, int n_targets, const double* target_xy,
                            const int32_t* center_index, double* out, hipStream_t stream) {
  if (n_ctr < 1 || n_targets < 0) return fail(QBX_EINVAL, "n_ctr = %d, n_targets = %d", n_ctr,
                                                n_targets);
  if (p < 0 || p > kPMax) return fail(QBX_EINVAL, "order p = %d outside [0, %d]", p, kPMax);
  if (!(k > 0.0) || !std::isfinite(k)) return fail(QBX_EINVAL, "wavenumber k = %g must be > 0", k);
  if (kind != QBX_S && kind != QBX_D && kind != (QBX_S | QBX_D))
    return fail(QBX_EINVAL, "kind = %d is not 1 (S), 2 (D) or 3 (S|D)", kind);
  if (n_targets == 0) return QBX_OK;
  if (!ctr_xy || !coef || !target_xy || !center_index || !out)
    return fail(QBX_EINVAL, "NULL array argument");
  const int nk = kind == 3 ? 2 : 1;
  hipLaunchKernelGGL(k_evaluate_expansions, dim3((n_targets + 255) / 256), dim3(256), 0, stream,
                     n_ctr, ctr_xy, reinterpret_cast<const double2*>(coef), k, p, nk, n_targets,
                     target_xy, center_index, reinterpret_cast<double2*>(out));
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? QBX_OK : device_fail(e, "expansion evaluation kernel");
}

int qbx_assign_centers(int n_ctr, const double* ctr_xy, const double* ctr_r, int n_targets,
                       const double* target_xy, double slack, int32_t* center_index,
                       hipStream_t stream) {
  if (n_ctr < 1 || n_targets < 0) return fail(QBX_EINVAL, "n_ctr = %d, n_targets = %d", n_ctr,
                                                n_targets);
  if (!(slack > 0.0) || !std::isfinite(slack))
    return fail(QBX_EINVAL, "slack = %g must be > 0", slack);
  if (n_targets == 0) return QBX_OK;
  if (!ctr_xy || !ctr_r || !target_xy || !center_index)
    return fail(QBX_EINVAL, "NULL array argument");
  // four targets a wave once that leaves enough waves to fill the device
  const int nt = n_targets >= 4096 ? 4 : 1;
  const dim3 grid((unsigned)(((long)n_targets + 4 * nt - 1) / (4 * nt)));
  if (nt == 4)
    hipLaunchKernelGGL(k_assign_centers<4>, grid, dim3(256), 0, stream, n_ctr, ctr_xy, ctr_r,
                       slack, n_targets, target_xy, center_index);
  else
    hipLaunchKernelGGL(k_assign_centers<1>, grid, dim3(256), 0, stream, n_ctr, ctr_xy, ctr_r,
                       slack, n_targets, target_xy, center_index);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? QBX_OK : device_fail(e, "center assignment kernel");
}

}  // extern "C"
