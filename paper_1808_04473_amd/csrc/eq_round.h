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
  float2 A[NS][UT][UT];  // swizzled rows (lds_el)
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

// Loads row i of system `sme` from LDS and factorises / solves it.
template <int UT>
struct FactorSolve {
  Factor<UT> f;
  float2 z;
  float d;
  float norm1;
  int fail;
  bool bad;
};

// PAD (factor_solve): leave out the steps of the factorisation and inverse
// that only touch padded users, for at most 24 users in a 32-lane group
// (PAD & 1) or 8 in a 16-lane group (PAD & 2); the FD forms, which solve one
// system per cluster, use it (PD measured no faster).
template <int UT, int PAD = 0, class SM>
__device__ __forceinline__ void factor_local(FactorSolve<UT> &r, SM &sm, int sme, int i, int U) {
  float rowsum = 0.f;
#pragma unroll
  for (int k = 0; k < UT; ++k) {
    r.f.a[k] = lds_el<UT>(sm.A[sme], i, k);
    rowsum = abs_row_acc(rowsum, r.f.a[k]);
  }
  const float2 m = sm.M[sme][i];
  r.bad = gany<UT>(!isfinite(abs_row_acc(rowsum, m)));
  r.norm1 = gmax<UT>(i < U ? rowsum * (1.f / kRowScale) : 0.f);
  // with fewer slots than groups (PD items of one 32-lane system) the freed
  // registers raise occupancy, so the inverse reads L from LDS there
  // with a slot per system, the 32 x 32 forms run their two block products
  // on MFMA through the slots (read above, free until the solve ends)
  float2 *split = nullptr;
  if constexpr (UT == 32 && SM::NS == SM::NSYS) split = &sm.A[0][0][0];
  r.z = factor_solve<UT, PAD>(r.f, i, m, r.fail, SM::NS < SM::NSYS ? sm.A[sme] : nullptr, split, U);
  r.d = inv_diag<UT>(r.f);
}

// LDS of one wave of the local solves: NSLOT packed matrix slots (one per
// system of a round by default; fewer when the work items hold fewer systems
// than there are lane groups) and, per system, every lane's share of the
// matched filter: 10 KB at 16 users, so 16 waves per CU, and 13 KB (12 waves)
// at 32.  R: right-hand sides of the refinement step.
template <int UT, int NS>
struct RefineRhs {
  float2 R[NS][UT];
};
struct NoRefineRhs {};
template <int UT, bool REFINE, int NSLOT = 64 / UT>
struct SolveSmem : std::conditional_t<REFINE, RefineRhs<UT, NSLOT>, NoRefineRhs> {
  static constexpr int NS = NSLOT;
  float2 A[NS * kSlot<UT>];
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
  Factor<UT> f;
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
