// Per-wave round state shared by the forward and backward kernels: the LDS
// staging of a round of NSYS = 64/UT small systems and the per-group
// factorisation of one system.
#pragma once
#include <type_traits>

#include "eq_device.h"

namespace dbpeq {

// NS matrix slots (one per system of a round by default; fewer when the
// work items hold fewer systems than there are lane groups, which leaves
// room for more waves per CU).
template <int UT, int NSLOT = 64 / UT>
struct Smem {
  static constexpr int NSYS = 64 / UT;
  static constexpr int NS = NSLOT;
  alignas(128) float2 A[NS][UT][UT];  // swizzled rows (lds_el)
  float2 M[NS][UT];
  float4 F[NS][UT];
  int routed[NSYS];
};

// LDS slot of lane group g: groups beyond the slots alias the last one (they
// then solve a copy of that system, and write nothing).
template <class SM>
__device__ __forceinline__ int slot_of(int g) {
  return g < SM::NS ? g : SM::NS - 1;
}

// LDS of one wave of the local solves: NSLOT packed matrix slots (one per
// system of a round by default; fewer when the work items hold fewer systems
// than there are lane groups) and, per system, every lane's share of the
// matched filter: 10 KB at 16 users, so 16 waves per CU, and 13.3 KB at 32 (11
// one-wave workgroups, 6 of two waves: LDS is given in units of 1,280 bytes).  R: right-hand sides of the refinement step.
template <int UT, int NS>
struct RefineRhs {
  float2 R[NS][UT];
};
struct NoRefineRhs {};
template <int UT, bool REFINE, int NSLOT = 64 / UT>
struct SolveSmem : std::conditional_t<REFINE, RefineRhs<UT, NSLOT>, NoRefineRhs> {
  static constexpr int NS = NSLOT;
  alignas(128) float2 A[NS * kSlot<UT>];  // GramAddr flips address bits below 128
  float2 M[NS][64];
};

// Factorises and solves the system of lane group `sme` (slot `sme`); KEEP
// leaves X = L^{-1} in the slot for the refinement step.
template <int UT, bool KEEP, class SM>
__device__ __forceinline__ void local_solve(LocalSolve<UT> &r, SM &sm, int sme, int i, float rho, int U) {
  float2 m = sm.M[sme][i];
#pragma unroll
  for (int g = 1; g < 64 / UT; g += 2) {
    const float2 p = sm.M[sme][g * UT + i];
    float2 q = make_float2(0.f, 0.f);
    if (g + 1 < 64 / UT) q = sm.M[sme][(g + 1) * UT + i];
    // (p0 + p1) + (p2 + p3)
    if (g == 1) m = make_float2(m.x + p.x, m.y + p.y);
    if (g + 1 < 64 / UT) {
      const float2 t = sm.M[sme][(g + 2) * UT + i];
      m = make_float2(m.x + (q.x + t.x), m.y + (q.y + t.y));
      break;
    }
  }
  solve_slot<UT, KEEP, SM::NS>(r, sm.A, sme, i, m, rho, U);
}

// Sum over the gw lane groups that share a subcarrier (gw = 1, 2, 4 groups,
// consecutive and aligned); every lane of them receives it.
template <int UT>
__device__ __forceinline__ float group_sum(float v, int gw) {
  if (UT == 16 && gw > 1) {
    const BSrc r = bsrc<32>(v);
    v = r.lo + r.hi;
  }
  if (gw > (UT == 16 ? 2 : 1)) v = xor32_sum(v);
  return v;
}

// One refinement step for the systems of a round: every group's z goes to
// LDS, the residual pass streams the systems' rows again and each group
// solves A dz = H^H (y - H z) - rho z as dz = X^H (X r) with X = L^{-1}
// (A^{-1} = X^H X): local_solve left X in the slot during the pass, t = X r
// is read along rows of X and dz = X^H t uses the columns.
template <int UT, class SM, class Rho, class Seg>
__device__ __forceinline__ void refine_round(LocalSolve<UT> &r, SM &sm, int nvalid, int U,
                                             Rho rhof, Seg seg, bool live) {
  const int lane = lane_id();
  const int sme = slot_of<SM>(lane / UT), i = lane % UT;
  wave_sync();
  sm.M[sme][i] = r.z;
  wave_sync();
  residual_stream<UT>(
      nvalid, U, seg, [&](int s) { return sm.M[s][lane % UT]; },
      [&](int s, float2 n) {
        const float2 zc = sm.M[s][lane % UT];
        const float rho = rhof(s);
        if (lane < UT) sm.R[s][lane] = make_float2(n.x - rho * zc.x, n.y - rho * zc.y);
      });
  wave_sync();
  float2 *As = sm.A + sme * kSlot<UT>;
  const int h = UT == 32 ? i >> 4 : 0, ii = i & 15;
  // t_j = sum_u X_ju r_u at lane j; the slot holds conj(X_ju) in row u
  float tx = 0.f, ty = 0.f;
  auto add = [&](float2 x, float2 rv) {
    tx = fmaf(x.x, rv.x, fmaf(x.y, rv.y, tx));
    ty = fmaf(x.x, rv.y, fmaf(-x.y, rv.x, ty));
  };
#pragma unroll
  for (int u = 0; u < 16; ++u) add(blk_el(As, h, u, ii), sm.R[sme][u]);
  if (UT == 32 && h) {
#pragma unroll
    for (int u = 0; u < 16; ++u) add(blk_el(As, 2, u, ii), sm.R[sme][16 + u]);
  }
  Columns<UT> f;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    float2 x = blk_el(As, 0, ii, k);
    if (h) x = make_float2(0.f, 0.f);
    f.x[k] = make_float2(x.x, -x.y);
    if constexpr (UT == 32) {
      x = blk_el(As, 1 + h, ii, k);
      f.x[16 + k] = make_float2(x.x, -x.y);
    }
  }
  const float2 dz = apply_xh<UT>(f, make_float2(tx, ty));
  if (live) {
    r.z.x += dz.x;
    r.z.y += dz.y;
  }
}

}  // namespace dbpeq
