// Adjoint kernels of libqbx: the forward-with-tape and source-major pair
// loops (bodies and derivations in qbx_pair.h), the per-center gradients from
// the tape, and the chain rule back to the 16-node panels.
#include "qbx_far.h"
#include "qbx_pair.h"
#include "qbx_panel.h"

namespace qbx {

// ---------------------------------------------------------------------------
// forward with tape (center-major, one wave per center and source split)
// partial layout: [n_tsplit][nk][Mc][5] complex = U, F_R, F_t, GV_x, GV_y
// ---------------------------------------------------------------------------
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_forward_tape(const double4* __restrict__ geo,
                                                      const double2* __restrict__ dens, int N,
                                                      const CenterRec* __restrict__ ctr,
                                                      const double* __restrict__ jtab, int NJ,
                                                      int Mc, int n_split, int chunks,
                                                      int chunks_per_split, double k,
                                                      double2* __restrict__ partial) {
  constexpr bool kS = (KIND & 1) != 0;
  constexpr bool kD = (KIND & 2) != 0;
  constexpr int NK = (kS ? 1 : 0) + (kD ? 1 : 0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + wave;
  const int ci = gw / n_split;
  const int sp = gw - ci * n_split;
  if (ci >= Mc) return;
  Cplx A[2][5];
  const int c0 = sp * chunks_per_split;
  const int c1 = min(c0 + chunks_per_split, chunks);
  tape_center<P, KIND>(geo, dens, N, ctr + ci, jtab + (size_t)ci * NJ, NJ, k, c0, c1, lane, A);
  if (lane == 0) {
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int b = 0; b < 5; ++b)
        partial[(((size_t)sp * NK + kk) * Mc + ci) * 5 + b] = make_double2(A[kk][b].r, A[kk][b].i);
  }
}

// out = (i/4) sum_splits U;  tape[ci][kk][0..3] = F_R, F_t, GV_x, GV_y
__global__ __launch_bounds__(256) void k_finalize_tape(int Mc, int T, int nk, int n_split,
                                                       const double2* __restrict__ partial,
                                                       double* __restrict__ out,
                                                       double2* __restrict__ tape) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Mc * nk) return;
  const int kk = e / Mc, ci = e - kk * Mc;
  double s[5][2] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}, {0, 0}};
  for (int sp = 0; sp < n_split; ++sp) {
    const double2* q = partial + (((size_t)sp * nk + kk) * Mc + ci) * 5;
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      s[b][0] += q[b].x;
      s[b][1] += q[b].y;
    }
  }
  const int si = ci / T, t = ci - si * T;
  if (out) {
    const size_t o = ((size_t)si * nk + kk) * T + t;
    out[2 * o] = -0.25 * s[0][1];
    out[2 * o + 1] = 0.25 * s[0][0];
  }
#pragma unroll
  for (int b = 0; b < 4; ++b)
    tape[((size_t)ci * nk + kk) * 4 + b] = make_double2(s[b + 1][0], s[b + 1][1]);
}

// ---------------------------------------------------------------------------
// target derivatives, pair pass: one wave per (center, source split), the
// launch shape of the tape pass; partial layout [n_split][nk][Mc][2] with
// q K_R and q K_theta summed over the split's sources
// ---------------------------------------------------------------------------
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_forward_grad(const double4* __restrict__ geo,
                                                      const double2* __restrict__ dens, int N,
                                                      const CenterRec* __restrict__ ctr,
                                                      const double* __restrict__ jtab, int NJ,
                                                      int Mc, int n_split, int chunks,
                                                      int chunks_per_split, double k,
                                                      double2* __restrict__ partial) {
  constexpr int NK = KIND == 3 ? 2 : 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + wave;
  const int ci = gw / n_split;
  const int sp = gw - ci * n_split;
  if (ci >= Mc) return;
  Cplx A[2][2];
  const int c0 = sp * chunks_per_split;
  const int c1 = min(c0 + chunks_per_split, chunks);
  // the order-weighted block follows the Mc tables (launch_order_weighted)
  grad_center<P, KIND>(geo, dens, N, ctr + ci, jtab + (size_t)ci * NJ, NJ,
                       jtab + (size_t)Mc * NJ + (size_t)ci * (NJ / 2), k, c0, c1, lane, A);
  if (lane == 0) {
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        partial[(((size_t)sp * NK + kk) * Mc + ci) * 2 + b] = make_double2(A[kk][b].r, A[kk][b].i);
  }
}

// ---------------------------------------------------------------------------
// target derivatives from the pair pass's partial sums (Section 3.2: the local
// expansion differentiated at the target).  With F_R = sum_j q_j dK/dR and
// F_t = sum_j q_j dK/dtheta (R, theta the target's polar coordinates about its
// center, w^ = e^{i theta}),
//   grad u = (i/4) (F_R w^ + (F_t / R) theta^),   n . grad u = -s (i/4) F_R,
// since the center lies at x + s R n (s = +1 exterior), so that w^ = -s n.
// grad: [n_sides][nk][T][2] complex; dn: [n_sides][nk][T] complex; either may
// be null.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_finalize_gradient(int Mc, int T, int nk, int n_split,
                                                           int side,
                                                           const CenterRec* __restrict__ ctr,
                                                           const double2* __restrict__ partial,
                                                           double* __restrict__ grad,
                                                           double* __restrict__ dn) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= Mc * nk) return;
  const int kk = e / Mc, ci = e - kk * Mc;
  double fr = 0.0, fi = 0.0, tr = 0.0, ti = 0.0;   // F_R, F_theta
  for (int sp = 0; sp < n_split; ++sp) {
    const double2* q = partial + (((size_t)sp * nk + kk) * Mc + ci) * 2;
    fr += q[0].x;
    fi += q[0].y;
    tr += q[1].x;
    ti += q[1].y;
  }
  const int si = ci / T, t = ci - si * T;
  const double s = side != 0 ? (double)side : (si == 0 ? 1.0 : -1.0);
  const size_t o = ((size_t)si * nk + kk) * T + t;
  // (i/4) z = (-Im z / 4, Re z / 4)
  if (dn) {
    dn[2 * o] = 0.25 * s * fi;
    dn[2 * o + 1] = -0.25 * s * fr;
  }
  if (grad) {
    const CenterRec c = ctr[ci];
    const double ir = 1.0 / c.R;
    // F_R w^ + (F_t / R) theta^, theta^ = (-sin, cos)
    const double gxr = fma(fr, c.ct, -tr * ir * c.st), gxi = fma(fi, c.ct, -ti * ir * c.st);
    const double gyr = fma(fr, c.st, tr * ir * c.ct), gyi = fma(fi, c.st, ti * ir * c.ct);
    double* q = grad + 4 * o;
    q[0] = -0.25 * gxi;
    q[1] = 0.25 * gxr;
    q[2] = -0.25 * gyi;
    q[3] = 0.25 * gyr;
  }
}

// ---------------------------------------------------------------------------
// G_i = conj(g_i) i/4 per center and kind: G[kk][ci]
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_make_G(int Mc, int T, int nk, const double* __restrict__ cot,
                                                double2* __restrict__ G) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < Mc * nk) make_G_elem(e, Mc, T, nk, cot, G);
}

// ---------------------------------------------------------------------------
// per-center gradients from the tape: cg[ci] = {g_x, g_y, g_R, g_nx, g_ny}
// (target position, panel-scaled radius R, target normal), before the chain rule
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_center_grads(int Mc, int nk, int side, int T,
                                                      const CenterRec* __restrict__ ctr,
                                                      const double2* __restrict__ tape,
                                                      const double2* __restrict__ G,
                                                      double* __restrict__ cg) {
  const int ci = blockIdx.x * blockDim.x + threadIdx.x;
  if (ci < Mc) center_grad_elem(ci, Mc, nk, side, T, ctr, tape, G, cg);
}

// ---------------------------------------------------------------------------
// source-major adjoint pass: one wave per (64 sources, center split), loop over
// centers; partial layout [n_csplit][src_slots(KIND)][N] (see src_slots)
// ---------------------------------------------------------------------------
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_adjoint_src(const double4* __restrict__ geo,
                                                     const double2* __restrict__ dens, int N,
                                                     const CenterRec* __restrict__ ctr,
                                                     const double* __restrict__ jtab, int NJ,
                                                     const double2* __restrict__ G, int Mc,
                                                     int n_csplit, int centers_per_split,
                                                     int chunks, double k,
                                                     double2* __restrict__ partial) {
  constexpr int NA = src_slots(KIND);
  constexpr int NK = KIND == 3 ? 2 : 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + wave;
  const int sb = gw / n_csplit;
  const int cs = gw - sb * n_csplit;
  if (sb >= chunks) return;
  const int j = sb * kWave + lane;
  if (j >= N) return;   // no cross-lane communication below
  const double4 g = geo[j];
  const int i0 = cs * centers_per_split;
  const int i1 = min(i0 + centers_per_split, Mc);
  double2 q[2];
  q[0] = dens[j];
  q[1] = dens[(size_t)(NK - 1) * N + j];
  Cplx A[NA];
  adjoint_source<P, KIND>(g, q, ctr, jtab, NJ, G, Mc, i0, i1, k, A);
#pragma unroll
  for (int b = 0; b < NA; ++b)
    partial[((size_t)cs * NA + b) * N + j] = make_double2(A[b].r, A[b].i);
}

// ---------------------------------------------------------------------------
// fused adjoint (no tape): one workgroup per tile (center block cb, source
// block sb); the tile body and its ordering are in qbx_pair.h (fused_tile)
// ---------------------------------------------------------------------------
template <int P, int KIND>
__global__ __launch_bounds__(256) void k_adjoint_fused(
    const double4* __restrict__ geo, const double2* __restrict__ dens, int N,
    const CenterRec* __restrict__ ctr, const double* __restrict__ jtab, int NJ,
    const double2* __restrict__ G, int Mc, int cblock, int n_sb, int chunks,
    int chunks_per_sb, double k, double2* __restrict__ spart, double* __restrict__ cpart) {
  constexpr int NA = src_slots(KIND);
  __shared__ double acc[4 * fused_centers(KIND) * 4];
  const int cb = blockIdx.x / n_sb;
  const int sb = blockIdx.x - cb * n_sb;
  const int i0 = cb * cblock;
  const int ch0 = sb * chunks_per_sb;
  fused_tile<P, KIND>(geo, dens, N, ctr, jtab, NJ, G, Mc, i0, min(cblock, Mc - i0), ch0,
                      min(ch0 + chunks_per_sb, chunks), k, spart + (size_t)cb * NA * N,
                      cpart + (size_t)sb * Mc * 4, acc);
}

// per center: the fused center-side sums over the source blocks, then the
// gradient assembly of center_grad_from_sums
__global__ __launch_bounds__(256) void k_fused_center_grads(int Mc, int n_sb, int side, int T,
                                                            const CenterRec* __restrict__ ctr,
                                                            const double* __restrict__ cpart,
                                                            double* __restrict__ cg) {
  const int ci = blockIdx.x * blockDim.x + threadIdx.x;
  if (ci >= Mc) return;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int sb = 0; sb < n_sb; ++sb) {
    const double* q = cpart + ((size_t)sb * Mc + ci) * 4;
#pragma unroll
    for (int b = 0; b < 4; ++b) s[b] += q[b];
  }
  center_grad_from_sums(ci, side, T, ctr, s[0], s[1], s[2], s[3], cg);
}

// 64 sources a block: the parts joined, then the gradients of source_grads_from_sums
__global__ __launch_bounds__(256) void k_source_finalize(int N, int kind, int n_csplit,
                                                         const FarItem* __restrict__ item,
                                                         const double4* __restrict__ geo,
                                                         const double2* __restrict__ partial,
                                                         double* __restrict__ sg) {
  double s[4][2] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
  int j;
  if (item && far_off(*item)) n_csplit = item->n_cb;
  if (join_source_parts(N, kind, n_csplit, partial, &j, s))
    source_grads_from_sums(j, kind, geo, s, sg);
}

__global__ __launch_bounds__(128) void k_chain(Dims d, const double* __restrict__ nodes,
                                               const double* __restrict__ density,
                                               const double* __restrict__ tab,
                                               const double* __restrict__ sg,
                                               const double* __restrict__ cg,
                                               const double* __restrict__ gtw,
                                               const double* __restrict__ gde,
                                               double* __restrict__ grad_density,
                                               double* __restrict__ grad_nodes) {
  chain_panel(d, blockIdx.x, nodes, density, tab, sg, cg, gtw, gde, grad_density, grad_nodes);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int P>
static hipError_t launch_forward_tape_p(const Dims& d, const double4* geo, const double2* dens,
                                        const CenterRec* ctr, const double* jtab,
                                        double2* partial, hipStream_t s) {
  const long waves = (long)d.Mc * d.n_tsplit;
  const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
#define QBX_LAUNCH(KD)                                                                          \
  hipLaunchKernelGGL((k_forward_tape<P, KD>), grid, block, 0, s, geo, dens, d.N, ctr, jtab, d.NJ, \
                     d.Mc, d.n_tsplit, d.chunks, d.tape_chunks_per_split, d.k, partial)
  if (d.kind == 1)
    QBX_LAUNCH(1);
  else if (d.kind == 2)
    QBX_LAUNCH(2);
  else
    QBX_LAUNCH(3);
#undef QBX_LAUNCH
  return hipGetLastError();
}

template <int P>
static hipError_t launch_adjoint_src_p(const Dims& d, const double4* geo, const double2* dens,
                                       const CenterRec* ctr, const double* jtab, const double2* G,
                                       double2* partial, hipStream_t s) {
  const long waves = (long)d.chunks * d.n_csplit;
  const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
#define QBX_LAUNCH(KD)                                                                       \
  hipLaunchKernelGGL((k_adjoint_src<P, KD>), grid, block, 0, s, geo, dens, d.N, ctr, jtab,    \
                     d.NJ, G, d.Mc, d.n_csplit, d.centers_per_split, d.chunks, d.k, partial)
  if (d.kind == 1)
    QBX_LAUNCH(1);
  else if (d.kind == 2)
    QBX_LAUNCH(2);
  else
    QBX_LAUNCH(3);
#undef QBX_LAUNCH
  return hipGetLastError();
}

hipError_t launch_forward_tape(const Dims& d, const double4* geo, const double2* dens,
                               const CenterRec* ctr, const double* jtab, double2* partial,
                               hipStream_t s) {
  QBX_P_SWITCH(d.p, launch_forward_tape_p, d, geo, dens, ctr, jtab, partial, s)
}

hipError_t launch_adjoint_src(const Dims& d, const double4* geo, const double2* dens,
                              const CenterRec* ctr, const double* jtab, const double2* G,
                              double2* partial, hipStream_t s) {
  QBX_P_SWITCH(d.p, launch_adjoint_src_p, d, geo, dens, ctr, jtab, G, partial, s)
}

hipError_t launch_finalize_tape(const Dims& d, const double2* partial, double* out, double2* tape,
                                hipStream_t s) {
  const int n = d.Mc * d.nk;
  hipLaunchKernelGGL(k_finalize_tape, dim3((n + 255) / 256), dim3(256), 0, s, d.Mc, d.T, d.nk,
                     d.n_tsplit, partial, out, tape);
  return hipGetLastError();
}

template <int P>
static hipError_t launch_forward_grad_p(const Dims& d, const double4* geo, const double2* dens,
                                       const CenterRec* ctr, const double* jtab,
                                       double2* partial, hipStream_t s) {
  const long waves = (long)d.Mc * d.n_tsplit;
  const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
#define QBX_LAUNCH(KD)                                                                          \
  hipLaunchKernelGGL((k_forward_grad<P, KD>), grid, block, 0, s, geo, dens, d.N, ctr, jtab, d.NJ, \
                     d.Mc, d.n_tsplit, d.chunks, d.tape_chunks_per_split, d.k, partial)
  if (d.kind == 1)
    QBX_LAUNCH(1);
  else if (d.kind == 2)
    QBX_LAUNCH(2);
  else
    QBX_LAUNCH(3);
#undef QBX_LAUNCH
  return hipGetLastError();
}

hipError_t launch_forward_grad(const Dims& d, const double4* geo, const double2* dens,
                               const CenterRec* ctr, const double* jtab, double2* partial,
                               hipStream_t s) {
  QBX_P_SWITCH(d.p, launch_forward_grad_p, d, geo, dens, ctr, jtab, partial, s)
}

hipError_t launch_finalize_gradient(const Dims& d, const CenterRec* ctr, const double2* partial,
                                    double* grad, double* dn, hipStream_t s) {
  const int n = d.Mc * d.nk;
  hipLaunchKernelGGL(k_finalize_gradient, dim3((n + 255) / 256), dim3(256), 0, s, d.Mc, d.T, d.nk,
                     d.n_tsplit, d.side, ctr, partial, grad, dn);
  return hipGetLastError();
}

template <int P>
static hipError_t launch_adjoint_fused_p(const Dims& d, const double4* geo, const double2* dens,
                                         const CenterRec* ctr, const double* jtab,
                                         const double2* G, double2* spart, double* cpart,
                                         hipStream_t s) {
  const dim3 grid((unsigned)(d.n_cb * d.n_sb)), block(256);
#define QBX_LAUNCH(KD)                                                                        \
  hipLaunchKernelGGL((k_adjoint_fused<P, KD>), grid, block, 0, s, geo, dens, d.N, ctr, jtab,   \
                     d.NJ, G, d.Mc, d.fused_cblock, d.n_sb, d.chunks, d.chunks_per_sb, d.k,    \
                     spart, cpart)
  if (d.kind == 1)
    QBX_LAUNCH(1);
  else if (d.kind == 2)
    QBX_LAUNCH(2);
  else
    QBX_LAUNCH(3);
#undef QBX_LAUNCH
  return hipGetLastError();
}

hipError_t launch_fused_tiles(const Dims& d, const double4* geo, const double2* dens,
                              const CenterRec* ctr, const double* jtab, const double2* G,
                              double2* spartial, double* cpart, hipStream_t s) {
  timer_begin(4, s);
  hipError_t e;
  switch (d.p) {
#define QBX_CASE(PP) \
  case PP:           \
    e = launch_adjoint_fused_p<PP>(d, geo, dens, ctr, jtab, G, spartial, cpart, s); \
    break;
    QBX_CASE(0) QBX_CASE(1) QBX_CASE(2) QBX_CASE(3) QBX_CASE(4) QBX_CASE(5) QBX_CASE(6)
    QBX_CASE(7) QBX_CASE(8) QBX_CASE(9) QBX_CASE(10) QBX_CASE(11) QBX_CASE(12) QBX_CASE(13)
    QBX_CASE(14) QBX_CASE(15) QBX_CASE(16) QBX_CASE(17) QBX_CASE(18) QBX_CASE(19) QBX_CASE(20)
    QBX_CASE(21) QBX_CASE(22) QBX_CASE(23) QBX_CASE(24)
#undef QBX_CASE
    default:
      e = hipErrorInvalidValue;
  }
  timer_end(4, s);
  return e;
}

hipError_t launch_adjoint_fused(const Dims& d, const double* nodes, const double* density,
                                const double* tables, const double4* geo, const double2* dens,
                                const CenterRec* ctr, const double* jtab, const double* cot,
                                double2* G, double* cpart, double* cg, double2* spartial,
                                double* sg, double* grad_density, double* grad_nodes,
                                hipStream_t s) {
  const int n = d.Mc * d.nk;
  hipLaunchKernelGGL(k_make_G, dim3((n + 255) / 256), dim3(256), 0, s, d.Mc, d.T, d.nk, cot, G);
  const hipError_t e = launch_fused_tiles(d, geo, dens, ctr, jtab, G, spartial, cpart, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fused_center_grads, dim3((d.Mc + 255) / 256), dim3(256), 0, s, d.Mc,
                     d.n_sb, d.side, d.T, ctr, cpart, cg);
  hipLaunchKernelGGL(k_source_finalize, dim3((d.N + kWave - 1) / kWave), dim3(256), 0, s, d.N, d.kind,
                     d.n_cb, nullptr, geo, spartial, sg);
  hipLaunchKernelGGL(k_chain, dim3(d.P), dim3(128), 0, s, d, nodes, density, tables, sg, cg,
                     nullptr, nullptr, grad_density, grad_nodes);
  return hipGetLastError();
}

hipError_t launch_chain(const Dims& d, const double* nodes, const double* density,
                        const double* tables, const double* sg, const double* cg,
                        const double* gtw, const double* gde, double* grad_density,
                        double* grad_nodes, hipStream_t s) {
  hipLaunchKernelGGL(k_chain, dim3(d.P), dim3(128), 0, s, d, nodes, density, tables, sg, cg,
                     gtw, gde, grad_density, grad_nodes);
  return hipGetLastError();
}

hipError_t launch_source_finalize(const Dims& d, int parts, const FarItem* item,
                                  const double4* geo, const double2* spart, double* sg,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_source_finalize, dim3((d.N + kWave - 1) / kWave), dim3(256), 0, s, d.N, d.kind,
                     parts, item, geo, spart, sg);
  return hipGetLastError();
}

hipError_t launch_make_G(const Dims& d, const double* cot, double2* G, hipStream_t s) {
  const int n = d.Mc * d.nk;
  hipLaunchKernelGGL(k_make_G, dim3((n + 255) / 256), dim3(256), 0, s, d.Mc, d.T, d.nk, cot, G);
  return hipGetLastError();
}

hipError_t launch_adjoint_rest(const Dims& d, const double* nodes, const double* density,
                               const double* tables, const double4* geo, const double2* dens,
                               const CenterRec* ctr, const double* jtab, const double* cot,
                               const double2* tape, double2* G, double* cg, double2* spartial,
                               double* sg, double* grad_density, double* grad_nodes,
                               hipStream_t s) {
  const int n = d.Mc * d.nk;
  hipLaunchKernelGGL(k_make_G, dim3((n + 255) / 256), dim3(256), 0, s, d.Mc, d.T, d.nk, cot, G);
  // without a tape only the density gradient is asked for (the node gradient
  // needs the center side): the chain step then reads no center data
  if (tape)
    hipLaunchKernelGGL(k_center_grads, dim3((d.Mc + 255) / 256), dim3(256), 0, s, d.Mc, d.nk,
                       d.side, d.T, ctr, tape, G, cg);
  timer_begin(1, s);
  hipError_t e = launch_adjoint_src(d, geo, dens, ctr, jtab, G, spartial, s);
  timer_end(1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_source_finalize, dim3((d.N + kWave - 1) / kWave), dim3(256), 0, s, d.N, d.kind,
                     d.n_csplit, nullptr, geo, spartial, sg);
  hipLaunchKernelGGL(k_chain, dim3(d.P), dim3(128), 0, s, d, nodes, density, tables, sg, cg,
                     nullptr, nullptr, grad_density, grad_nodes);
  return hipGetLastError();
}

}  // namespace qbx
