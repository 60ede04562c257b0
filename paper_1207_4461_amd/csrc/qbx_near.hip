// Near pairs: the pairs of a center and a source that are evaluated one by one when
// the far ones are summed otherwise (the panel expansions of qbx_far.hip, the direct rule
// of the near/far split).  One wave per center, or per 64 sources of a panel, walks its
// panel's near list; panels with more than kNearCap near panels are served by a scan of
// all panels.  The pair bodies are those of the plain
// kernels (qbx_pair.h).
#include "qbx_near.h"
#include "qbx_pair.h"
#include "qbx_panel.h"

// compiled once per kind, so that the template instances build in parallel
#ifndef QBX_NEAR_KIND
#error "compile with -DQBX_NEAR_KIND=1, 2 or 3"
#endif

namespace qbx {

// v[0..2 N) of every wave's lane 0 added in wave order into the first's
template <int N>
__device__ __forceinline__ void join_waves(double* v, int wave, int lane) {
  __shared__ double part[4][2 * N];
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) part[wave][i] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2 * N; ++i)
    v[i] = ((part[0][i] + part[1][i]) + part[2][i]) + part[3][i];
}

// Values.  Plain: out = (i/4) (near + far), the far sums of k_far_eval; split: the near
// sums alone into partial[kk][ci] (its finalize adds the far rule's).
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_near_forward(FarBlocks B, const double* __restrict__ ro,
                                                      double* __restrict__ wo,
                                                      double* __restrict__ out) {
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool quad = it.quad && far_off(it);
  const int ci = quad ? b : b * 4 + wave;
  if (ci >= it.Mc) return;
  const int first = quad ? wave * kWave : 0, step = quad ? 4 * kWave : kWave;
  const int m = (ci % it.T) / kQ;                 // the target's panel
  const double4* __restrict__ geo = reinterpret_cast<const double4*>(ro + it.geo);
  const double2* __restrict__ dens = reinterpret_cast<const double2*>(ro + it.dens);
  const CenterRec* C = reinterpret_cast<const CenterRec*>(ro + it.ctr) + ci;
  const double cx = C->cx, cy = C->cy, ct = C->ct, st = C->st;
  const double k = it.k, inv_k = 1.0 / k;
  const int N = it.N, qs = it.qs;
  const double* Jtab = ro + it.jtab + (size_t)ci * it.NJ;
  double sr = 0.0, si = 0.0, dr = 0.0, di = 0.0;
  for_near_runs(m, near_rel(it, ro), it.P, near_lists(it, ro), lane, [&](int pan, int n) {
    for (int s0 = first; s0 < n * qs; s0 += step) {
      if (s0 + lane < n * qs)
        forward_source<P, KIND>(geo, dens, N, pan * qs + s0 + lane, cx, cy, ct, st, k, inv_k,
                                Jtab, sr, si, dr, di);
    }
  });
  Cplx S = {sr, si}, Dd = {k * dr, k * di};
  if (kS) wave_sum(S);
  if (kD) wave_sum(Dd);
  Cplx v[2];
  v[0] = kS ? S : Dd;
  v[1] = Dd;
  if (quad) join_waves<2>(&v[0].r, wave, lane);
  if (lane == 0 && !(quad && wave > 0)) {
    if (it.pt) {
      double2* partial = reinterpret_cast<double2*>(wo + it.partial);
#pragma unroll
      for (int kk = 0; kk < NK; ++kk)
        partial[(size_t)kk * it.Mc + ci] = make_double2(v[kk].r, v[kk].i);
    } else {
      const double2* fu = reinterpret_cast<const double2*>(ro + it.fu);
      const bool add = !far_off(it);
      const int s = ci / it.T, t = ci - s * it.T;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        const double2 f = add ? fu[(size_t)kk * it.Mc + ci] : make_double2(0.0, 0.0);
        double* o = out + it.out_off + 2 * (((size_t)s * NK + kk) * it.T + t);
        o[0] = -0.25 * (v[kk].i + f.y);   // (i/4)(near + far)
        o[1] = 0.25 * (v[kk].r + f.x);
      }
    }
  }
}

// Target derivatives: partial[kk][ci][0..1] = F_R, F_theta over the near sources; plain:
// with the far ones.
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_near_grad(FarBlocks B, const double* __restrict__ ro,
                                                   double* __restrict__ wo) {
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool quad = it.quad && far_off(it);
  const int ci = quad ? b : b * 4 + wave;
  const int Mc = it.Mc, NJ = it.NJ;
  if (ci >= Mc) return;
  const int first = quad ? wave * kWave : 0, step = quad ? 4 * kWave : kWave;
  const int m = (ci % it.T) / kQ;
  const double4* __restrict__ geo = reinterpret_cast<const double4*>(ro + it.geo);
  const double2* __restrict__ dens = reinterpret_cast<const double2*>(ro + it.dens);
  const CenterRec* C = reinterpret_cast<const CenterRec*>(ro + it.ctr) + ci;
  const double cx = C->cx, cy = C->cy, ct = C->ct, st = C->st;
  const double k = it.k, inv_k = 1.0 / k;
  const int N = it.N, qs = it.qs;
  const double* Jtab = ro + it.jtab + (size_t)ci * NJ;
  const double* Ltab = ro + it.jtab + (size_t)Mc * NJ + (size_t)ci * (NJ / 2);   // l J_l
  Cplx A[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a) A[a][0] = A[a][1] = {0.0, 0.0};
  for_near_runs(m, near_rel(it, ro), it.P, near_lists(it, ro), lane, [&](int pan, int n) {
    for (int s0 = first; s0 < n * qs; s0 += step) {
      if (s0 + lane < n * qs)
        grad_source<P, KIND>(geo, dens, N, pan * qs + s0 + lane, cx, cy, ct, st, k, inv_k, Jtab,
                             NJ / 2, Ltab, A);
    }
  });
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    wave_sum(A[kk][0]);
    wave_sum(A[kk][1]);
  }
  if (quad) join_waves<4>(&A[0][0].r, wave, lane);
  if (lane == 0 && !(quad && wave > 0)) {
    const bool add = !it.pt && !far_off(it);
    const double2* fu = reinterpret_cast<const double2*>(ro + it.fu);
    double2* partial = reinterpret_cast<double2*>(wo + it.partial);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const size_t o = ((size_t)kk * Mc + ci) * 2 + q;
        const double2 f = add ? fu[o] : make_double2(0.0, 0.0);
        partial[o] = make_double2(A[kk][q].r + f.x, A[kk][q].i + f.y);
      }
  }
}

// A source pass's wave: share sp of ns of the list of chunk (panel, sub), 64 sources of one
// panel (fewer in the last)
struct NearChunk {
  int panel, sub, sp;
  bool on;
};
__device__ __forceinline__ NearChunk near_chunk(const FarItem& it, int w) {
  NearChunk c;
  const int subs = near_subs(it.qs), ns = it.nsrc;
  const int ch = w / ns;
  c.sp = w - ch * ns;
  c.panel = ch / subs;
  c.sub = ch - c.panel * subs;
  c.on = c.panel < it.P;
  return c;
}

// A share's part of the centers of the panels on a chunk's list, in sixteenths of a panel's
// centers: contiguous ranges, equal to one sixteenth.  (Whole panels dealt in turn, 13 to 8
// shares, left five with twice the work of the others: 1024 panels, p = 16, S: 349 us, 307 so.)
struct CenterShare {
  int lo, hi, at;
  __device__ __forceinline__ CenterShare(const NearChunk& c, const FarItem& it, int n_near) {
    const long long units = (long long)n_near * kQ;
    lo = (int)(units * c.sp / it.nsrc);
    hi = (int)(units * (c.sp + 1) / it.nsrc);
    at = 0;
  }
  // the part [c0, c1) of the next panel's nc centers; false: none
  __device__ __forceinline__ bool next(int nc, int* c0, int* c1) {
    const int a = max(lo - at, 0), b = min(hi - at, kQ);
    at += kQ;
    *c0 = a * (nc / kQ);
    *c1 = b * (nc / kQ);
    return a < b;
  }
};

// Adjoint, one evaluation per near pair (fused_pair) for both gradient sides.  Lanes are
// the sources of a chunk; the wave walks its share of the panel's near list and the
// centers of each panel on it.
//  * source side, in the lanes: spart[sp][b][j], b < src_slots(KIND); plain: the first
//    share adds the far sums (fs).
//  * center side: four reals a pair, summed over the lanes (the reduce-scatter of
//    fused_tile) into LDS and from there into the chunk's slot of the target panel,
//    cpart[panel][slot][center][4], slot = position of the chunk's panel in the target
//    panel's list (times the chunks of a panel).  Panels whose list is longer than
//    the item's slots have none: k_near_centers sums their centers.
// Replaces a pass per side (1758 and 1259 flops a pair at p = 20, S + D) by one of 1432.
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_near_sources(FarBlocks B, const double* __restrict__ ro,
                                                      double* __restrict__ wo) {
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = kS && kD ? 2 : 1;
  constexpr int NA = src_slots(KIND);
  __shared__ double csum[4][2 * kQ * 4];
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (!it.pt && far_off(it)) return;   // k_near_tiles
  const NearChunk c = near_chunk(it, b * 4 + wave);
  if (!c.on) return;
  const int N = it.N, qs = it.qs, T = it.T, Mc = it.Mc, NJ = it.NJ;
  const bool valid = c.sub * kWave + lane < qs;
  const int j = c.panel * qs + (valid ? c.sub * kWave + lane : qs - 1);
  const double4* __restrict__ geo = reinterpret_cast<const double4*>(ro + it.geo);
  const double2* __restrict__ dens = reinterpret_cast<const double2*>(ro + it.dens);
  const CenterRec* __restrict__ ctr = reinterpret_cast<const CenterRec*>(ro + it.ctr);
  const double* __restrict__ jtab = ro + it.jtab;
  const double2* __restrict__ G = reinterpret_cast<const double2*>(ro + it.G);
  const double4 g = geo[j];
  double2 q[2];   // lanes past the panel's sources take part in the sums with zeros
  q[0] = valid ? dens[j] : make_double2(0.0, 0.0);
  q[1] = NK == 2 && valid ? dens[(size_t)N + j] : make_double2(0.0, 0.0);
  const double k = it.k, inv_k = 1.0 / k;
  const int nj = NJ / 2, nc = it.n_sides * kQ;
  const int subs = near_subs(qs);
  const NearLists nl = near_lists(it, ro);
  double* __restrict__ cs = csum[wave];
  Cplx A[NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) A[a] = {0.0, 0.0};
  CenterShare share(c, it, nl.count[c.panel]);
  for_near_panels(c.panel, near_rel(it, ro), it.P, nl, lane, [&](int m) {
    int c0, c1;
    if (!share.next(nc, &c0, &c1)) return;
    const int cnt = nl.count[m];
    for (int cc = c0; cc < c1; ++cc) {
      const int si = cc / kQ;
      const int ci = si * T + m * kQ + (cc - si * kQ);
      const int z0 = opaque_zero();
      const CenterRec* __restrict__ C = ctr + ci + z0;
      double2 Gk[2];
      Gk[0] = G[(size_t)ci + z0];
      Gk[1] = NK == 2 ? G[(size_t)Mc + ci + z0] : Gk[0];
      double cres[4];
      fused_pair<P, KIND>(g, q, C->cx, C->cy, C->ct, C->st, jtab + (size_t)ci * NJ + z0, nj,
                          g_seed_table + z0, k, inv_k, Gk, A, cres);
      const double v = wave_sum4(cres, lane);
      if ((lane & 15) == 0) cs[cc * 4 + (lane >> 4)] = v;
    }
    if (cnt <= it.slots) {
      const int* __restrict__ L = nl.list + (size_t)m * kNearCap;
      // (the relation is symmetric, so the panel is on the list)
      int pos = 0;
      for (int i = 0; i < cnt; i += kWave) {
        const unsigned long long at =
            __ballot(i + lane < cnt && L[i + lane < cnt ? i + lane : 0] == c.panel);
        if (at) pos = i + __builtin_ctzll(at);
      }
      const int slot = pos * subs + c.sub;
      double* __restrict__ o =
          wo + it.cpart + (((size_t)m * it.slots * subs + slot) * nc) * 4;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      for (int t = 4 * c0 + lane; t < 4 * c1; t += kWave) o[t] = cs[t];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  });
  if (valid) {
    double2* part = reinterpret_cast<double2*>(wo + it.spart) + (size_t)c.sp * NA * N;
    const double2* fs = reinterpret_cast<const double2*>(ro + it.fs);
    const bool add = c.sp == 0 && !it.pt;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const double2 f = add ? fs[(size_t)a * N + j] : make_double2(0.0, 0.0);
      part[(size_t)a * N + j] = make_double2(A[a].r + f.x, A[a].i + f.y);
    }
  }
}

// Adjoint, center side of panels with slots: the slots in list order, plain: after the far
// sums (fc); four lanes a center, then center_grad_from_sums.  With the expansions off: the
// fused tiles' sums of every center.
template <int KIND>
__global__ __launch_bounds__(256) void k_near_center_sums(FarBlocks B,
                                                          const double* __restrict__ ro,
                                                          double* __restrict__ wo) {
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int e = b * 256 + threadIdx.x;
  const int ci = e >> 2, q = e & 3;
  if (ci >= it.Mc) return;   // whole groups of four lanes
  const int si = ci / it.T, t = ci - si * it.T;
  const int m = t / kQ;
  double s = 0.0;
  if (!it.pt && far_off(it)) {
    const double* __restrict__ p = ro + it.tpart + (size_t)ci * 4 + q;
    for (int sb = 0; sb < it.n_sb; ++sb) s += p[(size_t)sb * it.Mc * 4];
  } else {
    const int cnt = near_lists(it, ro).count[m];
    if (cnt > it.slots) return;
    const int subs = near_subs(it.qs), nc = it.n_sides * kQ;
    const double* __restrict__ p =
        ro + it.cpart + ((size_t)m * it.slots * subs * nc + si * kQ + (t - m * kQ)) * 4 + q;
    if (!it.pt) s = ro[it.fc + (size_t)ci * 4 + q];
    for (int i = 0; i < cnt * subs; ++i) s += p[(size_t)i * nc * 4];
  }
  const int l0 = threadIdx.x & ~3;
  const double s0 = __shfl(s, (l0 & 63)), s1 = __shfl(s, (l0 & 63) + 1),
               s2 = __shfl(s, (l0 & 63) + 2), s3 = __shfl(s, (l0 & 63) + 3);
  if (q == 0)
    center_grad_from_sums(ci, it.side, it.T, reinterpret_cast<const CenterRec*>(ro + it.ctr), s0,
                          s1, s2, s3, wo + it.cg);
}

// Adjoint, center side of panels without slots, one wave a center: the tape sums over the near
// sources (K_R, K_theta, grad_v K) contracted with G, plain: plus the far ones (fc).
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_near_centers(FarBlocks B, const double* __restrict__ ro,
                                                      double* __restrict__ wo) {
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int ci = b * 4 + wave;
  const int Mc = it.Mc;
  if (ci >= Mc) return;
  if (!it.pt && far_off(it)) return;   // k_near_center_sums
  const int m = (ci % it.T) / kQ;
  if (near_lists(it, ro).count[m] <= it.slots) return;
  const double4* __restrict__ geo = reinterpret_cast<const double4*>(ro + it.geo);
  const double2* __restrict__ dens = reinterpret_cast<const double2*>(ro + it.dens);
  const CenterRec* ctr = reinterpret_cast<const CenterRec*>(ro + it.ctr);
  const CenterRec* C = ctr + ci;
  const double cx = C->cx, cy = C->cy, ct = C->ct, st = C->st;
  const double k = it.k, inv_k = 1.0 / k;
  const int N = it.N, qs = it.qs;
  const double* Jtab = ro + it.jtab + (size_t)ci * it.NJ;
  const int nj = it.NJ / 2;
  Cplx A[2][5];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int q = 0; q < 5; ++q) A[a][q] = {0.0, 0.0};
  for_near_panels(m, near_rel(it, ro), it.P, near_lists(it, ro), lane, [&](int pan) {
    for (int s0 = 0; s0 < qs; s0 += kWave) {
      if (s0 + lane < qs)
        tape_source<P, KIND>(geo, dens, N, pan * qs + s0 + lane, cx, cy, ct, st, k, inv_k, Jtab,
                             nj, A);
    }
  });
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)
#pragma unroll
    for (int q = 1; q < 5; ++q) wave_sum(A[kk][q]);
  if (lane == 0) {
    const double2* G = reinterpret_cast<const double2*>(ro + it.G);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (!it.pt) {
      const double* fc = ro + it.fc + (size_t)ci * 4;
#pragma unroll
      for (int q = 0; q < 4; ++q) s[q] = fc[q];
    }
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const double2 g = G[(size_t)kk * Mc + ci];
#pragma unroll
      for (int q = 0; q < 4; ++q) s[q] += g.x * A[kk][q + 1].r - g.y * A[kk][q + 1].i;   // Re(G a)
    }
    center_grad_from_sums(ci, it.side, it.T, ctr, s[0], s[1], s[2], s[3], wo + it.cg);
  }
}

// Adjoint with respect to the density alone: sum_i G_i K_ij over the near centers, into
// spart[sp][kk][j]; plain: conjugated and with the far sums (fs), as the source passes
// keep it.
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_near_density(FarBlocks B, const double* __restrict__ ro,
                                                      double* __restrict__ wo) {
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NA = src_slots(KIND);
  int b;
  const FarItem& it = *far_item(B, blockIdx.x, &b);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const NearChunk c = near_chunk(it, b * 4 + wave);
  if (!c.on) return;
  const int N = it.N, qs = it.qs, T = it.T, Mc = it.Mc, NJ = it.NJ;
  const bool valid = c.sub * kWave + lane < qs;
  const int j = c.panel * qs + (valid ? c.sub * kWave + lane : qs - 1);
  const CenterRec* __restrict__ ctr = reinterpret_cast<const CenterRec*>(ro + it.ctr);
  const double* __restrict__ jtab = ro + it.jtab;
  const double2* __restrict__ G = reinterpret_cast<const double2*>(ro + it.G);
  const double4 g = reinterpret_cast<const double4*>(ro + it.geo)[j];
  const double k = it.k, inv_k = 1.0 / k;
  const int n_sides = it.n_sides;
  double sr = 0.0, si = 0.0, dr = 0.0, di = 0.0;
  const NearLists nl = near_lists(it, ro);
  const NearRel R = near_rel(it, ro);
  CenterShare share(c, it, R.all ? it.P : nl.count[c.panel]);
  for_near_runs(c.panel, R, it.P, nl, lane, [&](int pan, int n) {
    for (int m = pan; m < pan + n; ++m) {
      int c0, c1;
      if (!share.next(n_sides * kQ, &c0, &c1)) continue;
      for (int cc = c0; cc < c1; ++cc) {
        const int si_ = cc / kQ;
        const int ci = si_ * T + m * kQ + (cc - si_ * kQ);
        const int z0 = opaque_zero();
        const double* __restrict__ J = jtab + (size_t)ci * NJ + z0;
        const double* __restrict__ cf = g_seed_table + z0;
        const CenterRec* C = ctr + ci;
        const double vx = g.x - C->cx, vy = g.y - C->cy;
        const double rho2 = fma(vx, vx, vy * vy);
        const double ir = rsqrt_refined(rho2);
        const double rho = rho2 * ir;
        const double cd = (C->ct * vx + C->st * vy) * ir;
        const double sd = (C->st * vx - C->ct * vy) * ir;
        double cps = 0.0, sps = 0.0;
        if (kD) {
          cps = C->ct * g.z + C->st * g.w;
          sps = C->st * g.z - C->ct * g.w;
        }
        double ks_r, ks_i, kd_r, kd_i;
        pair_kernel<P, KIND>(k * rho, ir * inv_k, cd, sd, cps, sps, J, cf, ks_r, ks_i, kd_r,
                             kd_i);
        int kk = 0;
        if (kS) {
          const double2 Gi = G[(size_t)(kk++) * Mc + ci];
          sr = fma(Gi.x, ks_r, fma(-Gi.y, ks_i, sr));
          si = fma(Gi.x, ks_i, fma(Gi.y, ks_r, si));
        }
        if (kD) {
          const double2 Gi = G[(size_t)kk * Mc + ci];
          dr = fma(Gi.x, kd_r, fma(-Gi.y, kd_i, dr));
          di = fma(Gi.x, kd_i, fma(Gi.y, kd_r, di));
        }
      }
    }
  });
  if (valid) {
    const bool plain = !it.pt, add = plain && c.sp == 0 && !far_off(it);
    // the split sums near parts itself, [kk][j]; plain parts lie in the source-pass layout
    double2* part = reinterpret_cast<double2*>(wo + it.spart) +
                    (size_t)c.sp * (plain ? NA : (kS && kD ? 2 : 1)) * N;
    const double2* fs = reinterpret_cast<const double2*>(ro + it.fs);
    const double sg = plain ? -1.0 : 1.0;
    int kk = 0;
    if (kS) {
      const double2 f = add ? fs[j] : make_double2(0.0, 0.0);
      part[j] = make_double2(sr + f.x, sg * si + f.y);
      ++kk;
    }
    if (kD) {
      const double2 f = add ? fs[(size_t)kk * N + j] : make_double2(0.0, 0.0);
      part[(size_t)kk * N + j] = make_double2(k * dr + f.x, sg * k * di + f.y);
    }
  }
}

// Adjoint of items whose expansions are off: the fused tiles over every pair (fused_tile, the
// parts and center sums of k_adjoint_fused), taken by resident blocks from the item's counter
// (1024 panels, p = 16, S: 14.1 ms; dealt out in turn 16.7).  One launch beside the near passes;
// where every item is resolved its blocks return after a look at each.  next: the items'
// next_tile (apart from the items, which stay readable by scalar loads).
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_near_tiles(const FarItem* __restrict__ items, int n,
                                                    int* __restrict__ next,
                                                    const double* __restrict__ ro,
                                                    double* __restrict__ wo) {
  constexpr int NA = src_slots(KIND);
  constexpr int kItemInts = sizeof(FarItem) / sizeof(int);
  __shared__ double acc[4 * fused_centers(KIND) * 4];
  __shared__ int s_tile;
  for (int i = 0; i < n; ++i) {
    const FarItem& it = items[i];
    if (!far_off(it)) continue;
    const int tiles = it.n_cb * it.n_sb;
    for (;;) {   // the counter passes the tile count: every block leaves
      if (threadIdx.x == 0) s_tile = atomicAdd(next + i * kItemInts, 1);
      __syncthreads();
      const int b = s_tile;
      __syncthreads();   // every thread has read s_tile before the next fetch
      if (b >= tiles) break;
      const int cb = b / it.n_sb, sb = b - cb * it.n_sb;
      const int i0 = cb * it.cblock, ch0 = sb * it.chunks_per_sb;
      fused_tile<P, KIND>(reinterpret_cast<const double4*>(ro + it.geo),
                          reinterpret_cast<const double2*>(ro + it.dens), it.N,
                          reinterpret_cast<const CenterRec*>(ro + it.ctr), ro + it.jtab, it.NJ,
                          reinterpret_cast<const double2*>(ro + it.G), it.Mc, i0,
                          min(it.cblock, it.Mc - i0), ch0,
                          min(ch0 + it.chunks_per_sb, it.chunks), it.k,
                          reinterpret_cast<double2*>(wo + it.spart) + (size_t)cb * NA * it.N,
                          wo + it.tpart + (size_t)sb * it.Mc * 4, acc);
    }
  }
}

#if QBX_NEAR_KIND == 3
// Stored near pairs of the combined field alpha S - D, each the average of the two one-sided
// limits: mat[(m cap + slot) 256 + 16 a + t], the weight of node a of the slot-th panel near
// panel m in the potential at target t of m.  A block per (m, slot): the waves evaluate 4
// targets each against 64 sources at a time, both sides' centers, then a thread per (t, a)
// folds in the source weights and the interpolation V from the nodes.  Formed once per solve
// (about 1.5 forward near passes), it turns a product's near pass into a read of 4 KB per
// pair of near panels.
template <int P>
__global__ __launch_bounds__(256) void k_near_matrix(FarBlocks B, const double* __restrict__ ro,
                                                     int cap, const double* __restrict__ V,
                                                     const double* __restrict__ wgt, double2 alpha,
                                                     double2* __restrict__ mat) {
  __shared__ double2 c[kQ][kWave + 1];
  const FarItem& it = *B.items;
  const int m = blockIdx.x / cap, slot = blockIdx.x - m * cap;
  const NearLists nl = near_lists(it, ro);
  if (slot >= nl.count[m]) return;
  const int pan = nl.list[(size_t)m * kNearCap + slot];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int t = threadIdx.x & 15, a = threadIdx.x >> 4;
  const double4* __restrict__ geo = reinterpret_cast<const double4*>(ro + it.geo);
  const CenterRec* __restrict__ ctr = reinterpret_cast<const CenterRec*>(ro + it.ctr);
  const double k = it.k, inv_k = 1.0 / k;
  double2 acc = make_double2(0.0, 0.0);
  for (int s0 = 0; s0 < it.qs; s0 += kWave) {
    const int ns = min(kWave, it.qs - s0);
    const int j = pan * it.qs + s0 + min(lane, ns - 1);
    const double4 g = geo[j];
    const double w = 0.125 * wgt[j];
    for (int tt = 4 * wave; tt < 4 * wave + 4; ++tt) {
      double sr = 0.0, si = 0.0, dr = 0.0, di = 0.0;
      for (int side = 0; side < 2; ++side) {
        const int ci = side * it.T + m * kQ + tt;
        const int z0 = opaque_zero();
        const CenterRec* __restrict__ C = ctr + ci + z0;
        const double ct = C->ct, st = C->st;
        const double vx = g.x - C->cx, vy = g.y - C->cy;
        const double rho2 = fma(vx, vx, vy * vy);
        const double ir = rsqrt_refined(rho2);
        const double cd = (ct * vx + st * vy) * ir;
        const double sd = (st * vx - ct * vy) * ir;
        const double cps = ct * g.z + st * g.w;
        const double sps = st * g.z - ct * g.w;
        double ar, ai, br, bi;
        pair_kernel<P, 3>(k * (rho2 * ir), ir * inv_k, cd, sd, cps, sps,
                          ro + it.jtab + (size_t)ci * it.NJ + z0, g_seed_table + z0, ar, ai, br,
                          bi);
        sr += ar;
        si += ai;
        dr += br;
        di += bi;
      }
      // (i/8) w (alpha S - k D)
      const double ur = fma(alpha.x, sr, fma(-alpha.y, si, -k * dr));
      const double ui = fma(alpha.x, si, fma(alpha.y, sr, -k * di));
      c[tt][lane] = make_double2(-w * ui, w * ur);
    }
    __syncthreads();
    for (int q = 0; q < ns; ++q) {
      const double v = V[(s0 + q) * kQ + a];
      acc.x = fma(v, c[t][q].x, acc.x);
      acc.y = fma(v, c[t][q].y, acc.y);
    }
    __syncthreads();
  }
  mat[(size_t)blockIdx.x * (kQ * kQ) + threadIdx.x] = acc;
}

template <int P>
static hipError_t launch_near_matrix_p(const FarItem* dev, int n_panels, int cap, const double* V,
                                       const double* wgt, double2 alpha, double* ws, double2* mat,
                                       hipStream_t s) {
  hipLaunchKernelGGL(k_near_matrix<P>, dim3((unsigned)n_panels * cap), dim3(256), 0, s,
                     FarBlocks{dev, nullptr, 1}, ws, cap, V, wgt, alpha, mat);
  return hipGetLastError();
}
hipError_t launch_near_matrix(int p, const FarItem* dev, int n_panels, int cap, const double* V,
                              const double* wgt, double2 alpha, double* ws, double2* mat,
                              hipStream_t s) {
  QBX_P_SWITCH(p, launch_near_matrix_p, dev, n_panels, cap, V, wgt, alpha, ws, mat, s)
}
#endif

template <int P, int KIND>
static hipError_t launch_near_pk(NearPass pass, const FarBlocks& B, int blocks, double* ws,
                                 double* out, hipStream_t s) {
  const dim3 grid((unsigned)blocks), block(256);
  switch (pass) {
    case kNearForward:
      hipLaunchKernelGGL((k_near_forward<P, KIND>), grid, block, 0, s, B, ws, ws, out);
      break;
    case kNearGradient:
      hipLaunchKernelGGL((k_near_grad<P, KIND>), grid, block, 0, s, B, ws, ws);
      break;
    case kNearCenters:
      hipLaunchKernelGGL((k_near_centers<P, KIND>), grid, block, 0, s, B, ws, ws);
      break;
    case kNearCenterSums:
      hipLaunchKernelGGL((k_near_center_sums<KIND>), grid, block, 0, s, B, ws, ws);
      break;
    case kNearSources:
      hipLaunchKernelGGL((k_near_sources<P, KIND>), grid, block, 0, s, B, ws, ws);
      break;
    case kNearDensity:
      hipLaunchKernelGGL((k_near_density<P, KIND>), grid, block, 0, s, B, ws, ws);
      break;
  }
  return hipGetLastError();
}

template <int P>
static hipError_t launch_near_p(NearPass pass, const FarBlocks& B, int blocks, double* ws,
                                double* out, hipStream_t s) {
  return launch_near_pk<P, QBX_NEAR_KIND>(pass, B, blocks, ws, out, s);
}

template <int P>
static hipError_t launch_tiles_p(FarItem* items, int n, int blocks, double* ws,
                                 hipStream_t s) {
  hipLaunchKernelGGL((k_near_tiles<P, QBX_NEAR_KIND>), dim3((unsigned)blocks), dim3(256), 0, s,
                     items, n, &items->next_tile, ws, ws);
  return hipGetLastError();
}

#define QBX_CAT2(a, b) a##b
#define QBX_CAT(a, b) QBX_CAT2(a, b)
hipError_t QBX_CAT(launch_near_, QBX_NEAR_KIND)(NearPass pass, int p, const FarBlocks& B,
                                                int blocks, double* ws, double* out,
                                                hipStream_t s) {
  QBX_P_SWITCH(p, launch_near_p, pass, B, blocks, ws, out, s)
}
hipError_t QBX_CAT(launch_tiles_, QBX_NEAR_KIND)(int p, FarItem* items, int n, int blocks,
                                                 double* ws, hipStream_t s) {
  QBX_P_SWITCH(p, launch_tiles_p, items, n, blocks, ws, s)
}

}  // namespace qbx
