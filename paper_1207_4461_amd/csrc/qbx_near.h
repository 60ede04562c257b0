// The near relation of a call's item and the walk over a panel's near panels, shared by the
// near pairs' passes (qbx_near.hip) and the stored expansions (qbx_expansions.hip).
#pragma once

#include "qbx_far.h"

namespace qbx {

// near relation of an item: the split's gamma relation, or every pair of panels that no
// expansion takes, every pair where the expansions are off; symmetric
struct NearRel {
  FarRel R;
  bool gamma, all;
};
__device__ __forceinline__ NearRel near_rel(const FarItem& it, const double* ro) {
  NearRel n;
  n.gamma = it.pt != 0;
  n.all = !n.gamma && far_off(it);
  n.R.r0 = reinterpret_cast<const FarRec*>(ro + it.rec0);
  n.R.r1 = it.C1 > 0 ? reinterpret_cast<const FarRec*>(ro + it.rec1) : nullptr;
  n.R.g = it.g;
  n.R.bnd = reinterpret_cast<const double4*>(ro + it.bnd);
  n.R.g2 = it.g2;
  return n;
}
__device__ __forceinline__ bool is_near(const NearRel& n, int a, int b) {
  if (n.gamma) return panels_near(n.R.bnd[a], n.R.bnd[b], n.R.g2);
  FarRel R = n.R;
  R.bnd = nullptr;
  return !far_panels(R, a, b);
}

__device__ __forceinline__ NearLists near_lists(const FarItem& it, const double* ro) {
  NearLists l;
  l.count = reinterpret_cast<const int*>(ro + it.ncount);
  l.list = reinterpret_cast<const int*>(ro + it.nlist);
  return l;
}

// f(pan, n) for runs of n consecutive panels near panel m (wave-uniform), in ascending order:
// the panels of m's list one by one when it fits, else the wave's scan of all NP panels, up to
// 64 a run (a copy of f each: with one copy for both the near passes took 5 to 10% longer)
template <typename F>
__device__ __forceinline__ void for_near_runs(int m, const NearRel& R, int NP, NearLists nl,
                                                int lane, F&& f) {
  const int cnt = R.all ? kNearCap + 1 : nl.count[m];
  if (cnt <= kNearCap) {
    const int* __restrict__ L = nl.list + (size_t)m * kNearCap;
    for (int i = 0; i < cnt; ++i) f(L[i], 1);
    return;
  }
  for (int w0 = 0; w0 < NP; w0 += kWave) {
    const int mp = w0 + lane;
    const bool nr = mp < NP && (R.all || is_near(R, m, mp));
    unsigned long long mask = __ballot(nr);
    while (mask) {
      const int b0 = __builtin_ctzll(mask);
      const unsigned long long gap = ~(mask >> b0);   // 0: all 64 panels
      const int n = gap ? __builtin_ctzll(gap) : kWave;
      mask = n + b0 < kWave ? mask >> (b0 + n) << (b0 + n) : 0;
      f(w0 + b0, n);
    }
  }
}

// f(pan) for every panel near panel m, where the expansions are on (through for_near_runs the
// near adjoint took 272 us at 1024 panels, p = 16, S; so 256)
template <typename F>
__device__ __forceinline__ void for_near_panels(int m, const NearRel& R, int NP, NearLists nl,
                                                int lane, F&& f) {
  const int cnt = nl.count[m];
  if (cnt <= kNearCap) {
    const int* __restrict__ L = nl.list + (size_t)m * kNearCap;
    for (int i = 0; i < cnt; ++i) f(L[i]);
    return;
  }
  for (int w0 = 0; w0 < NP; w0 += kWave) {
    const int mp = w0 + lane;
    const bool nr = mp < NP && is_near(R, m, mp);
    unsigned long long mask = __ballot(nr);
    while (mask) {
      const int pan = w0 + __builtin_ctzll(mask);
      mask &= mask - 1;
      f(pan);
    }
  }
}

}  // namespace qbx
