// Far sums of the pair kernels through panel expansions: shared declarations of
// qbx_far.hip (the expansions) and qbx_near.hip (the pairs that stay pairs).
//
// The truncated expansion of Section 2 at a center c is linear in the field of the
// sources near c: its coefficients a_n, |n| <= p, are those of the local expansion of
// that field about c.  For a source panel far from a target panel that field is
// smooth, and three exact translations (Graf's addition theorem, eq. graf-addition)
// carry it from the sources of the one to the centers of the other at a cost per pair
// of panels instead of per pair of points:
//
//   M_m = sum_j q_j J_m(k r_j) e^{-i m alpha_j}        about the source panel's mean b_A,
//   L_l = sum_A sum_m M_m F_{m-l}(b_B - b_A)           F_n(D) = H_n(k|D|) e^{i n arg D},
//   a_n = sum_l L_l J_{l-n}(k|tau|) e^{i(l-n) arg tau}  tau = c - b_B,
//
// and the value is sum_n a_n J_n(k R) e^{i n theta} over |n| <= p, the truncation of
// the pair kernels.  The double layer takes the normal derivative of the regular
// waves in M_m.  Orders |m|, |l| <= kFarQ are kept; two panels are taken this way only
// where the terms beyond are below 1e-17 of the leading one (far_adm), so that the
// sums differ from the pair sums by rounding.  The same holds for groups of consecutive
// panels (FarItem::g), which take the pairs of groups that are far enough as one pair.
// Every other pair of panels is near, and its pairs are evaluated one by one.
//
// The adjoint is the transpose: T_l = sum_c G_c E_l(c) over the centers of a panel
// (E_l the value of the wave l at the center's target), carried by the same
// translation to the source panels, where the field's value and derivatives at each
// source are its gradients.
#pragma once

#include "qbx_internal.h"

namespace qbx {

constexpr int kFarQ = 24;        // order of the expansions
constexpr int kFarW = 2 * kFarQ + 1;

// One cluster (a panel or a group): mean of its nodes, radius of its sources (rs) and
// of its centers with their disks (rt), the distances from which an expansion of order
// kFarQ resolves them (ds, dt), and, for the near/far split's
// groups, the radius of the panel means (rb) and gamma times the largest node radius
// (gr): groups at least that far hold no pair of panels within gamma radii.
// Where the coefficients are the result, the distances are those that keep every order right
// (qbx_coef_table.h) and rt is the radius of the centers alone.
struct FarRec {
  double bx, by, rs, rt, ds, dt, rb, gr;
};

// Symmetric in its arguments bit for bit (no contraction; maxima and sums of two), so
// every kernel and both directions take the same decision.  False for NaN positions.
__device__ __forceinline__ bool far_adm(const FarRec& a, const FarRec& b) {
#pragma clang fp contract(off)
  const double dx = a.bx - b.bx, dy = a.by - b.by;
  const double d2 = dx * dx + dy * dy;
  const double t0 = fmax(fmax(a.ds + b.rt, b.ds + a.rt), fmax(a.dt + b.rs, b.dt + a.rs));
  const double t = fmax(t0, (a.rb + b.rb) + fmax(a.gr, b.gr));
  return d2 >= t * t;
}

// gamma relation of the near/far split (qbx_split.hip): every operation rounded on
// its own, the same decision for any IEEE evaluation of the formula
__device__ __forceinline__ bool panels_near(double4 a, double4 b, double g2) {
#pragma clang fp contract(off)
  const double dx = a.x - b.x;
  const double dy = a.y - b.y;
  const double d2 = dx * dx + dy * dy;
  return d2 < g2 * fmax(a.z, b.z);
}

// Which pairs of panels go through expansions: the pairs of far groups at once, the
// remaining far pairs of panels one by one.  With the gamma relation (bnd set) only
// pairs that it calls far.
struct FarRel {
  const FarRec* r0;    // panels
  const FarRec* r1;    // groups of g panels, or null
  int g;
  const double4* bnd;  // gamma relation's panels, or null
  double g2;
};
__device__ __forceinline__ bool far_panels(const FarRel& R, int a, int b) {
  if (R.r1 && far_adm(R.r1[a / R.g], R.r1[b / R.g])) return true;
  if (R.bnd && panels_near(R.bnd[a], R.bnd[b], R.g2)) return false;
  return far_adm(R.r0[a], R.r0[b]);
}

// One contour of a call.  Offsets count doubles from the workspace base.  Every call writes its
// items anew; in heavy and next_tile (0 then) its kernels leave what the later ones decide by.
struct FarItem {
  int P, C1, g;         // panels, groups (0: none), panels of a group (4 or 8)
  int T, N, qs, Mc, n_sides, nk, kind, p, NJ, side;
  int fqs;              // far sources per panel (qs; the split: 16, the nodes)
  int pt;               // the near/far split's item: far targets are points (its nodes), near
                        // pairs those of the gamma relation (at any gamma: g2 may underflow to 0)
  int coef;             // order of the coefficients that the call returns, or -1 (it sums them)
  int V;                // vectors translated: kinds forward, then kinds backward
  int vf;               // of them forward (0 or nk)
  int n_cb, n_sb, cblock, chunks, chunks_per_sb;   // the fused tiles (k_near_tiles)
  unsigned long long heavy;   // near panels of the panels with many, added up (k_far_lists)
  int next_tile;        // of the fused tiles
  double off_pairs;     // the sum from which the expansions are off (far_off)
  int slots;            // longest near list whose panel's center sums go through cpart
  int quad;             // with the expansions off, a block per center in the near passes over
                        // centers (a contour whose waves would not fill the GPU)
  int nsrc;             // waves per 64-source chunk in the near source passes
  int n0, n1;           // blocks of sources per 64 target panels / groups
  int m2l_blocks;       // translation blocks aimed for
  double k, g2;         // g2: the split's gamma squared
  size_t node_off;      // doubles into the nodes
  size_t out_off;       // doubles into out
  size_t geo, dens, ctr, jtab, G;      // pair sources, centers, cotangent weights
  size_t fgeo, fdens, fG;              // far sources and far targets' weights
  size_t bnd, rec0, rec1;
  size_t ncount, nlist;                // near lists: int arrays (still offsets in doubles)
  size_t mcount, mlist;                // lists of the panels no expansion takes (plain: the same)
  size_t rows0, rows1;                 // double2 [V][2][C][kFarW]
  size_t lp0, lp1;                     // double2 [n][V][2][kFarQ + 1][C]
  size_t ls0, ls1;                     // double2 [V][C][kFarW]
  size_t tp0, tp1;                     // double2 [n_sides or n_sides g / 4][nk][C][kFarW]
  size_t fu;                           // double2 [nk][Mc][2] far sums per center
  size_t fc;                           // double [Mc][4] far center gradients
  size_t fs;                           // double2 [nk + 2][far sources]
  size_t cpart;                        // double [P][slots subs][n_sides kQ][4]: near center sums
  size_t partial, cg, spart;           // near outputs: gradient sums, center / source gradients
  size_t tpart;                        // double [n_sb][Mc][4]: the fused tiles' center sums
};

// Expansions of one order do not resolve every contour: past k rt = 3.4 (about k h = 2.8 at
// r = 0.5), and at the other end where the contour is smaller than 1e-3 / k, every panel is
// near.  The host does not know the panels' sizes, so the lists decide on the device: where
// the near lists hold off_pairs pairs of panels, the expansions' kernels return at once, and
//  * forward, target derivatives, density adjoint and coefficients (from 0.9 P^2: translations
//    for a few lanes each cost what the pairs do): the near passes take every pair, in one run;
//  * the adjoint for the nodes, whose near passes evaluate the pairs of a panel twice when its
//    list is longer than its slots (from 0.4 P^2; 0.5 where the slots hold half the panels):
//    the fused tiles take every pair (k_near_tiles) and the near passes return too;
//  * the near/far split (from 0.3 P^2): its direct far passes, which share a panel's pairs out
//    over many waves, take the far pairs in place of k_split_mid.
// 1024 panels, S, p = 16, k = 900, in ms, before the expansions / with them and without this
// rule / now: forward 7.55 / 7.96 / 7.31, adjoint 14.4 / 30.7 / 14.1, split 0.71 / 2.28 /
// 0.71, split's adjoint 2.08 / 4.59 / 1.88.  What it costs a resolved contour: 1 to 3 us a
// forward, 5 to 10 an adjoint or a split (launches that return at once).
//
// Contours below kFarQuadCenters centers: one wave a center is too few (130 panels, S + D, p = 8,
// k = 200: near pass 225 us, a block a center 167, the pair loop's split waves 151).
constexpr int kFarQuadCenters = 8192;
// Blocks of k_near_tiles, which takes tiles from a counter: what is resident (at most five on each
// of 256 compute units).  A block per tile costs a resolved contour of 256 panels 16 us of 490,
// these 6.
constexpr int kFarTileBlocks = 1280;
constexpr double kFarOffPass = 0.9, kFarOffAdjoint = 0.4, kFarOffAdjointSmall = 0.5,
                 kFarOffSplit = 0.3;
__device__ __forceinline__ bool far_off(const FarItem& it) {
  return (double)it.heavy >= it.off_pairs;
}
// a panel whose list counts towards that: more than a quarter of the panels (13 to 15 are near
// where the expansions resolve the contour), so that the common case adds nothing
__device__ __forceinline__ bool far_heavy(int near, int P) { return 4 * (long long)near > P; }

// item of a block: prefix sums of the items' block counts, or a single item
struct FarBlocks {
  const FarItem* items;
  const int* pre;   // null: one item
  int n;
};
__device__ __forceinline__ const FarItem* far_item(const FarBlocks& B, int block, int* local) {
  int s = 0;
  if (B.pre) {
    int hi = B.n;   // pre[s] <= block < pre[hi]
    while (hi - s > 1) {
      const int mid = (s + hi) >> 1;
      if (B.pre[mid] <= block) s = mid;
      else hi = mid;
    }
    block -= B.pre[s];
  }
  *local = block;
  return B.items + s;
}

// the grids of the steps, per item
enum FarStep {
  kStepClusters,   // panels and groups, one wave each
  kStepM2L, kStepM2LGroups, kStepSum,
  kStepTargets,    // 64 targets of one side
  kStepRows, kStepSources, kStepLists,
  kStepCenters,    // four centers, one wave each (qbx_near.hip)
  kStepNear,       // the same, or a block per center (quad)
  kStepChunks,     // four shares of the chunks of 64 sources of a panel (qbx_near.hip)
  kStepCenterSums, // 64 centers, four lanes each (qbx_near.hip)
};
int far_blocks(const FarItem& it, FarStep step);

// the near pairs' passes (qbx_near.hip); out: kNearForward's result
// kNearCenterSums, kNearCenters: the two halves of the center side (short and long lists)
enum NearPass {
  kNearForward, kNearGradient, kNearSources, kNearCenterSums, kNearCenters, kNearDensity
};
// the fused tiles of those of the n items whose expansions are off, dealt out to `blocks` blocks
hipError_t launch_near_tiles(int p, int kind, FarItem* items, int n, int blocks, double* ws,
                             hipStream_t s);
// the near pairs of alpha S - D (two-sided averages) as matrices over the nodes of near
// panels, mat[P][cap][16 nodes][16 targets]; item dev with near lists, both sides and kinds
hipError_t launch_near_matrix(int p, const FarItem* dev, int n_panels, int cap, const double* V,
                              const double* wgt, double2 alpha, double* ws, double2* mat,
                              hipStream_t s);
hipError_t launch_near(NearPass pass, int p, int kind, const FarBlocks& B, int blocks,
                       double* ws, double* out, hipStream_t s);

// Blocks of the translation that are resident at once (256 compute units, three each), and the
// most shares of the sources a panel-level block takes when groups serve the rest (about 110
// sources are left per 64 target panels).
constexpr int kFarM2LBlocks = 768;
constexpr int kFarMaxPanelShares = 16;

// A call's items on the device and the grids of its steps.  One contour: the item in the
// workspace and no prefix arrays; a batch: every step's prefix sums of block counts.
struct FarPlan {
  FarBlocks at[kStepLists + 1];
  int blocks[kStepLists + 1];
};
// the plan of one item (device copy at `dev`)
FarPlan far_single(const FarItem& it, const FarItem* dev);
// records and near lists, multipoles (fwd) and their transpose (bwd), translations, and
// what the caller wants of them: values or sums at the targets (eval: the mode of
// launch_far_eval, or -1), gradients at the sources (src; geom: position and normal too)
hipError_t far_fields(const FarPlan& P, const double* nodes, double* ws, bool fwd, bool bwd,
                      int eval, bool src, bool geom, bool lists, hipStream_t s,
                      double2* coef = nullptr);
// the offsets of an item's far arrays from take(bytes) (returning a byte offset), with
// bwd those of the adjoint too; V, n0, n1 are then set per call (far_shape).  n_items: the
// items that share the call's launches; m2l_blocks: the translation blocks of a single item, fewer
// where their partial sums would not fit.
template <typename Take>
inline void far_layout(const Dims& d, bool bwd, Take&& take, FarItem* it, int n_items = 1,
                       int m2l_blocks = kFarM2LBlocks);
// vectors, translation shares and off_pairs of a call: fwd / bwd as in far_fields
void far_shape(FarItem* it, bool fwd, bool bwd);

hipError_t launch_far_recs(const FarBlocks& B, int blocks, const double* nodes, double* ws,
                           hipStream_t s);
hipError_t launch_far_lists(const FarBlocks& B, int blocks, double* ws, hipStream_t s);
hipError_t launch_far_p2m(const FarBlocks& B, int blocks, double* ws, hipStream_t s);
hipError_t launch_far_m2l(bool groups, const FarBlocks& B, int blocks, double* ws, hipStream_t s);
hipError_t launch_far_lsum(const FarBlocks& B, int blocks, double* ws, hipStream_t s);
// mode 0 values, 1 target derivatives, 2 center gradients contracted with G, 3 the coefficients
// of the centers (into coef)
hipError_t launch_far_eval(int mode, const FarBlocks& B, int blocks, double* ws, double2* coef,
                           hipStream_t s);
hipError_t launch_far_t(const FarBlocks& B, int blocks, double* ws, hipStream_t s);
hipError_t launch_far_rows(const FarBlocks& B, int blocks, double* ws, hipStream_t s);
hipError_t launch_far_src(const FarBlocks& B, int blocks, double* ws, bool geom, hipStream_t s);


// Near adjoint: a source panel's chunks of 64 (one partial), and the near lists up to which the
// fused pass also forms the center side (13 panels are near at most sizes; past them the centers
// of a panel are summed by a wave each, a second evaluation of every pair).  Small contours
// have room for more: at a few panels a wavelength, up to all 100 panels are near, and the
// second evaluation made batches of a few such contours slower than the pair tiles.
constexpr int kNearSlots = 32, kNearSlotsSmall = 128, kNearSlotsSmallPanels = 256;
static_assert(kNearSlotsSmall <= kNearCap, "slots are positions in the near lists");
__host__ __device__ inline int near_subs(int qs) { return (qs + kWave - 1) / kWave; }

// Where expansions take the far pairs.  A center distance r over 1 (a disk that reaches over
// many panels) leaves every panel near; below that what they save has to pay for their six
// launches and short chains (about 100 us in a forward, 220 in an adjoint, with both kinds
// 125 and 290), so a plain pass takes them from kFarMinPanels panels and from a forward pair
// count of kFarMinFlops (1 + kinds) on.  Forward, far / pair by pair in us: 96 panels, S,
// p = 4, q_s = 48: 104 / 68, 160 panels: 108 / 127; S, p = 8, q_s = 64, 112 panels: 109 / 108;
// S + D, p = 8, one side, 96 and 112 panels: 125 / 111, 126 / 143; both sides, p = 12, 96
// panels: 149 / 220.  Adjoint of the same: 220 / 131, 236 / 238, 239 / 211, 288 / 256,
// 285 / 322, 437 / 494.
// Others: a batch's contours share the launches; the split's direct far pairs are cheap, but its
// near passes came to the same walk (forward, S, p = 4: 64 panels 77, 96 panels 102, 128
// panels 106 us); the coefficients have a rule of
// their own (far_coef_size); a solve forms what it stores once.
constexpr int kFarMinPanels = 96, kFarMinCoefPanels = 16, kFarMinSolvePanels = 64;
constexpr int kFarMaxCoefOrder = 12;   // rows of qbx_coef_table.h
constexpr double kFarMinFlops = 1.4e9;
// From kFarGroupPanels panels on groups of four too, from kFarGroup8Panels on of eight.  The
// second level costs its own multipoles, sums and evaluation (about 70 us at 256 panels,
// where it saves less: forward 289 us without, 354 us with groups; at 333 panels 449 and
// 419 us), so a contour alone takes it later than one of a batch, whose items fill the
// GPU together (64 contours of 16..512 panels: translations 9.9 ms without, 2.6 ms with).
constexpr int kFarGroupPanels = 320, kFarGroupPanelsBatch = 128;
constexpr int kFarGroup8Panels = 2048;
inline bool far_fits(const Dims& d) { return d.center_rule == 0 && d.r <= 1.0; }
// flops of a forward over every pair
inline double pair_work(const Dims& d) {
  const double pair = d.kind == 1 ? 95 + 12 * d.p : d.kind == 2 ? 114 + 16 * d.p : 128 + 23 * d.p;
  return pair * d.Mc * d.N;
}
inline bool far_applies(const Dims& d) {
  return d.P >= kFarMinPanels && far_fits(d) && pair_work(d) >= kFarMinFlops * (1 + d.nk);
}
// A contour of a batch whose forward over every pair takes `work` flops.  Small batches do not
// fill the GPU, and the chain of launches and the few waves of a contour of 100 to 160 panels
// take longer than its pair tiles beside the others (forward and adjoint of 7 contours of up
// to 120 panels, 10 GFLOP: up to 2.7 ms by expansions, 2.2 ms without).
constexpr double kFarBatchFlops = 2e10;
inline bool far_applies_batch(const Dims& d, double work) {
  return d.P >= (work < kFarBatchFlops ? 160 : kFarMinPanels) && far_fits(d);
}
// Coefficients: near are 11 panels at p = 0, 23 at 6, 72 at 12 (qbx_coef_table.h), every one past
// that.  The near pass splits its pairs over more waves than the one over all pairs: 8 panels,
// S, p = 12: 139 us near, 103 all; 16 panels 113, 252; 256 panels 501, 2484; S + D, both sides,
// 256 panels 1754, 4365.  Where every panel is near that ends with the size: p = 24, one side,
// 256 panels 1732, 3396, 512 panels 6605, 6442; both sides 150 panels 3568, 4513, 256 panels
// 7428, 7377.
constexpr int kFarMaxAllNear = 320;    // panels times sides
inline bool far_coef_size(const Dims& d) {
  return d.P >= kFarMinCoefPanels &&
         (d.p <= kFarMaxCoefOrder || d.P * d.n_sides <= kFarMaxAllNear);
}
inline bool far_applies_coef(const Dims& d) { return far_coef_size(d) && far_fits(d); }
inline bool far_applies_solve(const Dims& d) { return d.P >= kFarMinSolvePanels && far_fits(d); }
// the near/far split's far targets are points: no disk to look at
inline bool far_applies_split(const Dims& d) { return d.P >= kFarMinPanels; }
// Waves of the near source passes aimed for, and parts of a chunk's near source sums at most; half
// of both in a batch, whose items fill the GPU together.  (8192 and 8, 16384 and 16: 1024
// panels, p = 16, S: near adjoint 307 and 288 us; 4096 panels, S + D: 3.97 and 3.87 ms; the
// batch of 64 contours: 12.5 and 12.7 ms.)
constexpr int kFarSourceWaves = 16384;
constexpr int kFarMaxShares = 16;
// Shares of the sources per (target block, vector, half): as many as `rounds` rounds of
// resident blocks hold, for the number of rounds that gives the least time (a partly
// filled last round costs a whole one); a batch's item: its part of four rounds.
inline int far_share(int C, int V, int blocks, bool inner) {
  const int base = (C + kWave - 1) / kWave * V * 2;
  int most = (C + 3) / 4, n = 1;
  if (inner && most > kFarMaxPanelShares) most = kFarMaxPanelShares;
  if (blocks < kFarM2LBlocks) {
    n = (blocks + base - 1) / base;
  } else {
    double best = 1e300;
    for (int rounds = 1; rounds <= 3; ++rounds) {
      int c = rounds * blocks / base;
      if (c < 1) continue;
      if (c > most) c = most;
      const int r = (c * base + blocks - 1) / blocks;
      if ((double)r / c < best * 0.999) {
        best = (double)r / c;
        n = c;
      }
    }
  }
  if (n > most) n = most;
  return n < 1 ? 1 : n;
}
inline size_t far_lp_doubles(int C, int Vmax, int blocks, bool inner) {
  size_t most = 0;   // over the vector counts a call may have
  for (int V = 1; V <= Vmax; ++V) {
    const size_t n = (size_t)far_share(C, V, blocks, inner) * V * 2 * (kFarQ + 1) * C * 2;
    if (n > most) most = n;
  }
  return most;
}

template <typename Take>
inline void far_layout(const Dims& d, bool bwd, Take&& take, FarItem* it, int n_items,
                       int m2l_blocks) {
  auto at = [&](size_t doubles) { return take(sizeof(double) * doubles) / sizeof(double); };
  *it = FarItem{};
  it->coef = -1;
  it->P = d.P;
  it->g = d.P >= kFarGroup8Panels ? 8 : 4;
  it->C1 = d.P >= (n_items > 1 ? kFarGroupPanelsBatch : kFarGroupPanels) ? (d.P + it->g - 1) / it->g : 0;
  it->T = d.T;
  it->N = d.N;
  it->qs = d.qs;
  it->fqs = d.qs;
  it->Mc = d.Mc;
  it->n_sides = d.n_sides;
  it->nk = d.nk;
  it->kind = d.kind;
  it->p = d.p;
  it->NJ = d.NJ;
  it->side = d.side;
  it->n_cb = d.n_cb;
  it->n_sb = d.n_sb;
  it->cblock = d.fused_cblock;
  it->chunks = d.chunks;
  it->chunks_per_sb = d.chunks_per_sb;
  const int Vmax = d.nk * (bwd ? 2 : 1);
  const size_t C0 = d.P, C1 = it->C1;
  it->rec0 = at(sizeof(FarRec) / sizeof(double) * C0);
  it->rec1 = at(sizeof(FarRec) / sizeof(double) * C1);
  it->ncount = it->mcount = at((C0 + 1) / 2);
  it->nlist = it->mlist = at(C0 * kNearCap / 2);
  it->rows0 = at((size_t)Vmax * 2 * C0 * kFarW * 2);
  it->rows1 = at((size_t)Vmax * 2 * C1 * kFarW * 2);
  // a batch's items share the GPU: four times a single item's blocks between them
  it->m2l_blocks = n_items > 1 ? (4 * kFarM2LBlocks + n_items - 1) / n_items : m2l_blocks;
  it->lp0 = at(far_lp_doubles(d.P, Vmax, it->m2l_blocks, it->C1 > 0));
  it->lp1 = at(it->C1 ? far_lp_doubles(it->C1, Vmax, it->m2l_blocks, false) : 0);
  it->ls0 = at((size_t)Vmax * C0 * kFarW * 2);
  it->ls1 = at((size_t)Vmax * C1 * kFarW * 2);
  it->fu = at((size_t)d.nk * d.Mc * (bwd ? 4 : 2));
  if (bwd) {
    it->tp0 = at((size_t)d.n_sides * d.nk * C0 * kFarW * 2);
    it->tp1 = at((size_t)(it->g / 4) * d.n_sides * d.nk * C1 * kFarW * 2);
    it->fc = at((size_t)d.Mc * 4);
    it->slots = d.P <= kNearSlotsSmallPanels ? kNearSlotsSmall : kNearSlots;
    it->cpart = at((size_t)it->slots * near_subs(d.qs) * d.Mc * 4);
    it->fs = at((size_t)(d.nk + 2) * d.N * 2);
  }
  it->quad = n_items == 1 && d.Mc < kFarQuadCenters;
  // a chunk's list is cut into at most kFarMaxShares
  const long long chunks = (long long)d.P * near_subs(d.qs) * n_items;
  const int waves = n_items > 1 ? kFarSourceWaves / 2 : kFarSourceWaves;
  const int most = n_items > 1 ? kFarMaxShares / 2 : kFarMaxShares;
  const int ns = (int)((waves + chunks - 1) / chunks);
  it->nsrc = ns > most ? most : ns;
}

}  // namespace qbx
