// Hand-written adjoint of the PD and FD L-MMSE equalisers (the paper gives
// the forward maps only; the derivation is in dbpeq.h and the FP64 oracle).
//
// For one system with A = G + rho I, z = A^{-1} y^MRC, d = diag(A^{-1}),
// upstream gradients gz (complex, of z) and gs (real, of sigma2 = N0 d):
//   lambda = A^{-1} gz,  Q = A^{-1} diag(gs) A^{-1},
//   grad_H = (y - H z) lambda^H - H K,  K = lambda z^H + 2 N0 Q,
//   grad_y = H lambda,
//   grad_N0 = -Re(z^H lambda)/E_s + sum_u gs_u d_u - N0 tr(Q)/E_s.
//
// A wave solves a round of systems (one per lane group) and leaves X = L^{-1}
// of each in LDS; then, system by system, the whole wave forms A^{-1} = X^H X
// and Q on MFMA.  Both come in accumulator layout, lane (kk, c) holding rows
// 4 kk + r of column c, and since A^{-1} is Hermitian its registers are their
// own A operand.  Last the rows are streamed again for grad_H and grad_y:
// lane (kk, c) loads the users 4 kk .. 4 kk + 3 of row c, which is the B
// operand of (H K)^T = K^T H^T, K's registers being the A operand, and the
// product comes back at the users and row the lane holds, to be written where
// it was read.
//
// PD treats each subcarrier as one system.  FD with optimal weights needs the
// sums S = sum_c p_c and sum_c p_c z_c (p_c = 1 / sigma2_c) of a subcarrier
// before any of its clusters can be differentiated: with nu_c = p_c / S and zb
// the fused estimate, the loss reaches sigma2_c through nu with
//   gs_c = gs nu_c^2 - p_c^2 Re(conj(gz) (z_c - zb)) / S
// (the terms of gs in dL/dnu_c are equal for every cluster and cancel).  One
// wave per round keeps its systems in LDS while the sums meet; subcarriers of
// more rounds than a workgroup has waves form every system twice.
#include "eq_round.h"

namespace dbpeq {

// ---------------------------------------------------------------- second pass over the rows
// 16 rows: row c of lane (kk, c), users 16 t + 4 kk + r in h[4 t + r].
template <int NT>
struct RowSlot {
  float2 h[4 * NT];
  float2 y;
  const float2 *Hw, *yw;
  int s, rb, r0, r1;
  bool first, last;
};

// QUAD: U is a multiple of 4, so a lane's four users are all real or all
// padding and 16-byte accesses are wholly inside or outside the descriptor.
template <int NT>
struct RowOff {
  unsigned h[4 * NT];  // h[4 t] with QUAD, every user without
  unsigned y;
};

template <int NT, bool QUAD>
__device__ __forceinline__ RowOff<NT> row_offsets(int U) {
  const int lane = lane_id();
  const int kk = lane / 16, c = lane % 16;
  RowOff<NT> o;
#pragma unroll
  for (int k = 0; k < 4 * NT; k += QUAD ? 4 : 1) {
    const int u = 16 * (k / 4) + 4 * kk + k % 4;
    o.h[k] = u < U ? (unsigned)((c * U + u) * 8) : kOutOfRange;
  }
  o.y = (unsigned)(c * 8);
  return o;
}

typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));

template <int NT, bool QUAD>
__device__ __forceinline__ void load_rows(RowSlot<NT> &b, const RowOff<NT> &o, int U, bool live) {
  const int nrow = live ? b.r1 - b.r0 : 0;
  const __amdgpu_buffer_rsrc_t rh =
      __builtin_amdgcn_make_buffer_rsrc((void *)(b.Hw + (size_t)b.r0 * U), (short)0, nrow * U * 8, kBufFlags);
  const __amdgpu_buffer_rsrc_t ry =
      __builtin_amdgcn_make_buffer_rsrc((void *)(b.yw + b.r0), (short)0, nrow * 8, kBufFlags);
  const unsigned rowb = (unsigned)((b.rb - b.r0) * U * 8);
#pragma unroll
  for (int k = 0; k < 4 * NT; k += 4) {
    if constexpr (QUAD) {
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        const f4 v = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rh, o.h[k] + rowb + 8u * j, 0, kLoadLast));
        b.h[k + j] = make_float2(v.x, v.y);
        b.h[k + j + 1] = make_float2(v.z, v.w);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) b.h[k + j] = buf_ld2<kLoadLast>(rh, o.h[k + j] + rowb);
    }
  }
  b.y = buf_ld2<kLoadLast>(ry, o.y + (unsigned)((b.rb - b.r0) * 8));
}

// Complex tile blocks in accumulator layout: block (a, b) holds rows 16 a + 4 kk
// + r, column 16 b + c.
template <int NT>
struct Blocks {
  f4 re[NT][NT], im[NT][NT];
};

// out += conj(a) b over k = (r, kk): with a's registers as the A operand
// [i = c][k], the rows of a are the k index (out = a^H b).
__device__ __forceinline__ void mul_hc(f4 &re, f4 &im, const f4 &ar, const f4 &ai, const f4 &br, const f4 &bi) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    re = mma32(ar[r], br[r], re);
    im = mma32(ar[r], bi[r], im);
    re = mma32(ai[r], bi[r], re);
    im = mma32(-ai[r], br[r], im);
  }
}

// A^{-1} = X^H X of slot As (conj(X_ku) in row u).
template <int NT>
__device__ __forceinline__ void ainv_blocks(float2 *As, Blocks<NT> &I) {
  const int lane = lane_id();
  const int kk = lane / 16, c = lane % 16;
  const f4 z0 = {0.f, 0.f, 0.f, 0.f};
  // x[b][r] = X_{16 e + 4 kk + r, 16 b + c} of row block e
  auto rows = [&](int blk, f4 &re, f4 &im) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float2 x = blk_el(As, blk, c, 4 * kk + r);
      re[r] = x.x;
      im[r] = -x.y;
    }
  };
  f4 xr, xi;
  rows(0, xr, xi);
  I.re[0][0] = I.im[0][0] = z0;
  mul_hc(I.re[0][0], I.im[0][0], xr, xi, xr, xi);
  if constexpr (NT == 2) {
    f4 wr, wi;
    rows(1, xr, xi);
    rows(2, wr, wi);
    mul_hc(I.re[0][0], I.im[0][0], xr, xi, xr, xi);
    I.re[0][1] = I.im[0][1] = I.re[1][0] = I.im[1][0] = I.re[1][1] = I.im[1][1] = z0;
    mul_hc(I.re[0][1], I.im[0][1], xr, xi, wr, wi);
    mul_hc(I.re[1][0], I.im[1][0], wr, wi, xr, xi);
    mul_hc(I.re[1][1], I.im[1][1], wr, wi, wr, wi);
  }
}

// LDS of one wave: X, then Q, of the round's systems; the matched-filter
// shares, then the fusion sums, then z (first UT entries) and lambda of each
// system.
template <int UT>
using BwdLds = SolveSmem<UT, false>;

// The second pass in the streaming layout, for gs = 0 and hence Q = 0: grad_H =
// (y - H z) lambda^H - (H lambda) z^H (stream_rows says where).
template <int UT, class Seg>
__device__ __forceinline__ void rank1_rows(const BwdArgs &a, BwdLds<UT> &sm, int nvalid, Seg seg) {
  const int lane = lane_id();
  const int col = lane % UT, g = lane / UT;
  const int U = a.U;
  float2 zc = sm.M[0][col], lc = sm.M[0][UT + col];
  stream_blocks<UT, kLoadLast>(
      nvalid, U, seg,
      [&](const Slot &b) {
        float2 *gHw = a.gH ? a.gH + (b.Hw - a.H) : nullptr;
        float2 *gyw = a.gy ? a.gy + (b.yw - a.y) : nullptr;
        sfor<8>([&](auto E) {
          constexpr int e = E;
          const float2 h = slot_h<UT>(b, e, U);
          const float hzx = gsum<UT>(h.x * zc.x - h.y * zc.y);
          const float hzy = gsum<UT>(h.x * zc.y + h.y * zc.x);
          const float hlx = gsum<UT>(h.x * lc.x - h.y * lc.y);
          const float hly = gsum<UT>(h.x * lc.y + h.y * lc.x);
          const float2 yv = slot_y<UT, e>(b);
          const float rx = yv.x - hzx, ry = yv.y - hzy;
          const int row = b.rb + slot_row(e, g);
          if (row < b.r1) {
            if (gHw && col < U)
              gHw[(size_t)row * U + col] = make_float2(rx * lc.x + ry * lc.y - (hlx * zc.x + hly * zc.y),
                                                       ry * lc.x - rx * lc.y - (hly * zc.x - hlx * zc.y));
            if (gyw && col == 0) gyw[row] = make_float2(hlx, hly);
          }
        });
      },
      [&](int s) {
        if (s + 1 < nvalid) {
          zc = sm.M[s + 1][col];
          lc = sm.M[s + 1][UT + col];
        }
      });
  wave_sync();
}

// Gradients of one round of systems, X in the slots of sm.  Lane (sme, i)
// holds the solve r and the upstream gradients gzc, gsc of user i of system
// sme.  Returns this lane's share of grad_N0.
template <int UT, bool QUAD, class Seg>
__device__ __forceinline__ float round_grads(const BwdArgs &a, BwdLds<UT> &sm, const LocalSolve<UT> &r, int nvalid,
                                             Seg seg, float2 gzc, float gsc) {
  constexpr int NT = UT / 16;
  const int lane = lane_id();
  const int kk = lane / 16, c = lane % 16;
  const int sme = lane / UT, i = lane % UT;
  const int U = a.U;
  const bool use_q = __ballot(gsc != 0.f) != 0ull;
  // value of user 16 t + 4 kk + r of system q
  auto user = [&](float v, int q, int t, int r4) { return __shfl(v, q * UT + 16 * t + 4 * kk + r4); };

  wave_sync();
  sm.M[sme][i] = r.z;
  // ---- lambda = X^H (X gz), every lane group its own system: t = X gz along the
  //      rows of X (lane k; the slot holds conj(X_ku) in row u), lambda along its
  //      columns (closer to the exact value than A^{-1} gz with A^{-1} formed)
  {
    float2 *As = sm.A + sme * kSlot<UT>;
    const int h = UT == 32 ? i >> 4 : 0, ii = i & 15;
    const BSrc gx = bsrc<UT>(gzc.x), gy = bsrc<UT>(gzc.y);
    float tx[2] = {0.f, 0.f}, ty[2] = {0.f, 0.f};
    sfor<UT>([&](auto Uu) {
      constexpr int u = Uu, p = u & 1;
      float2 x = blk_el(As, u < 16 ? h : 2, u & 15, ii);
      if (UT == 32 && u >= 16 && h == 0) x = make_float2(0.f, 0.f);
      const float bx = dpp<DPP_ROW_NEWBCAST + u % 16>(bpick<u>(gx)), by = dpp<DPP_ROW_NEWBCAST + u % 16>(bpick<u>(gy));
      tx[p] = fmaf(x.x, bx, fmaf(x.y, by, tx[p]));
      ty[p] = fmaf(x.x, by, fmaf(-x.y, bx, ty[p]));
    });
    const BSrc sx = bsrc<UT>(tx[0] + tx[1]), sy = bsrc<UT>(ty[0] + ty[1]);
    float lx[2] = {0.f, 0.f}, ly[2] = {0.f, 0.f};
    sfor<UT>([&](auto Kk) {
      constexpr int k = Kk, p = k & 1;
      float2 x = blk_el(As, k < 16 ? 0 : 1 + h, ii, k & 15);
      if (UT == 32 && k < 16 && h == 1) x = make_float2(0.f, 0.f);
      const float bx = dpp<DPP_ROW_NEWBCAST + k % 16>(bpick<k>(sx)), by = dpp<DPP_ROW_NEWBCAST + k % 16>(bpick<k>(sy));
      lx[p] = fmaf(x.x, bx, fmaf(-x.y, by, lx[p]));
      ly[p] = fmaf(x.x, by, fmaf(x.y, bx, ly[p]));
    });
    sm.M[sme][UT + i] = make_float2(lx[0] + lx[1], ly[0] + ly[1]);
  }
  // ---- Q, system by system
  for (int q = 0; use_q && q < nvalid; ++q) {
    float2 *As = sm.A + q * kSlot<UT>;
    Blocks<NT> I;
    ainv_blocks<NT>(As, I);
    // Q = A^{-1} (diag(gs) A^{-1}); A^{-1} is Hermitian, so a^H b it is
    f4 gsv[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int k = 0; k < 4; ++k) gsv[t][k] = user(gsc, q, t, k);
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      f4 wr[NT], wi[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        wr[t] = gsv[t] * I.re[t][b];
        wi[t] = gsv[t] * I.im[t][b];
      }
#pragma unroll
      for (int e = b; e < NT; ++e) {
        f4 re = {0.f, 0.f, 0.f, 0.f}, im = re;
#pragma unroll
        for (int t = 0; t < NT; ++t) mul_hc(re, im, I.re[t][e], I.im[t][e], wr[t], wi[t]);
#pragma unroll
        for (int k = 0; k < 4; ++k) blk_el(As, e + b, 4 * kk + k, c) = make_float2(re[k], im[k]);
      }
    }
  }
  wave_sync();
  float gn0 = 0.f;
  if (sme < nvalid && i < U) {
    const float2 lam = sm.M[sme][UT + i];
    const float inv_es = 1.0f / a.es;
    gn0 = -(r.z.x * lam.x + r.z.y * lam.y) * inv_es + gsc * r.d;
    if (use_q) gn0 -= a.n0 * blk_el(sm.A + sme * kSlot<UT>, i < 16 ? 0 : 2, i & 15, i & 15).x * inv_es;
  }

  // ---- the rows again: grad_H and grad_y
  if (!use_q && a.stream_rows) {
    rank1_rows<UT>(a, sm, nvalid, seg);
    return gn0;
  }
  const RowOff<NT> off = row_offsets<NT, QUAD>(U);
  SysRef cur;
  int next = 0;
  auto advance = [&]() {
    seg(next, cur.Hw, cur.yw, cur.r0, cur.r1);
    cur.s = next++;
  };
  advance();
  int crb = cur.r0;
  bool more = true;
  auto issue = [&](RowSlot<NT> &sl) -> bool {
    const bool valid = more;
    sl.Hw = cur.Hw;
    sl.yw = cur.yw;
    sl.rb = crb;
    sl.r0 = cur.r0;
    sl.r1 = cur.r1;
    sl.s = cur.s;
    sl.first = crb == cur.r0;
    sl.last = false;
    load_rows<NT, QUAD>(sl, off, U, valid);
    if (valid) {
      if (crb + 16 < cur.r1) {
        crb += 16;
      } else if (next < nvalid) {
        advance();
        crb = cur.r0;
      } else {
        more = false;
      }
    }
    return valid;
  };
  Blocks<NT> K;
  float2 zt[4 * NT], lt[4 * NT];
  auto body = [&](const RowSlot<NT> &b) {
    if (b.first) {
      // z, lambda of this lane's users, and K_{16 t + 4 kk + k, 16 b + c}
      float2 *As = sm.A + b.s * kSlot<UT>;
#pragma unroll
      for (int k = 0; k < 4 * NT; ++k) {
        const int u = 16 * (k / 4) + 4 * kk + k % 4;
        zt[k] = sm.M[b.s][u];
        lt[k] = sm.M[b.s][UT + u];
      }
      if (use_q) {
        const float n2 = 2.f * a.n0;
#pragma unroll
        for (int e = 0; e < NT; ++e) {
          const float2 zc = sm.M[b.s][16 * e + c];
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const float2 l = lt[4 * t + k];
              // block (0, 1) of Q is the conjugate transpose of (1, 0)
              const float2 qv = t >= e ? blk_el(As, t + e, 4 * kk + k, c) : blk_el(As, 1, c, 4 * kk + k);
              K.re[t][e][k] = fmaf(n2, qv.x, l.x * zc.x + l.y * zc.y);
              K.im[t][e][k] = fmaf(t >= e ? n2 : -n2, qv.y, l.y * zc.x - l.x * zc.y);
            }
        }
      }
    }
    // (H z), (H lambda) of row c
    float hzx = 0.f, hzy = 0.f, hlx = 0.f, hly = 0.f;
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) {
      const float2 h = b.h[k];
      hzx = fmaf(h.x, zt[k].x, fmaf(-h.y, zt[k].y, hzx));
      hzy = fmaf(h.x, zt[k].y, fmaf(h.y, zt[k].x, hzy));
      hlx = fmaf(h.x, lt[k].x, fmaf(-h.y, lt[k].y, hlx));
      hly = fmaf(h.x, lt[k].y, fmaf(h.y, lt[k].x, hly));
    }
    hzx = groups_sum(hzx);
    hzy = groups_sum(hzy);
    hlx = groups_sum(hlx);
    hly = groups_sum(hly);
    const float rx = b.y.x - hzx, ry = b.y.y - hzy;
    const int nrow = b.r1 - b.r0;
    const unsigned rowb = (unsigned)((b.rb - b.r0) * U * 8);
    if (a.gH) {
      const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
          (void *)(a.gH + (b.Hw - a.H) + (size_t)b.r0 * U), (short)0, nrow * U * 8, kBufFlags);
#pragma unroll
      for (int e = 0; e < NT; ++e) {
        // (H K)_{row c, 16 e + 4 kk + k}; without Q it is (H lambda) z^H
        f4 pr = {0.f, 0.f, 0.f, 0.f}, pi = pr;
        if (use_q) {
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const float2 h = b.h[4 * t + k];
              pr = mma32(K.re[t][e][k], h.x, pr);
              pi = mma32(K.re[t][e][k], h.y, pi);
              pr = mma32(-K.im[t][e][k], h.y, pr);
              pi = mma32(K.im[t][e][k], h.x, pi);
            }
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float2 z = zt[4 * e + k];
            pr[k] = hlx * z.x + hly * z.y;
            pi[k] = hly * z.x - hlx * z.y;
          }
        }
        float2 g[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float2 l = lt[4 * e + k];
          g[k] = make_float2(rx * l.x + ry * l.y - pr[k], ry * l.x - rx * l.y - pi[k]);
        }
        if constexpr (QUAD) {
#pragma unroll
          for (int k = 0; k < 4; k += 2) {
            const f4 v = {g[k].x, g[k].y, g[k + 1].x, g[k + 1].y};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), rg, off.h[4 * e] + rowb + 8u * k, 0, 0);
          }
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, g[k]), rg, off.h[4 * e + k] + rowb, 0, 0);
        }
      }
    }
    if (a.gy && kk == 0) {
      const int row = b.rb + c;
      if (row < b.r1) a.gy[(b.yw - a.y) + row] = make_float2(hlx, hly);
    }
  };
  auto done = [](const RowSlot<NT> &) {};
  stream_ring3<RowSlot<NT>>(issue, body, done);
  wave_sync();
  return gn0;
}

// Gram, matched filter and solve of a round's systems; X is left in the slots.
template <int UT, class Seg>
__device__ __forceinline__ void round_solve(const BwdArgs &a, BwdLds<UT> &sm, LocalSolve<UT> &r, int nvalid, Seg seg) {
  const int lane = lane_id();
  const GramAddr<UT> ga = gram_addr<UT>();
  gram_stream<UT, PREC_FP32, kLoadKeep>(nvalid, a.U, seg, [&](int s, const Acc<UT> &acc, float2 mf) {
    store_gram_packed<UT, PREC_FP32>(ga, sm.A + s * kSlot<UT>, acc);
    sm.M[s][lane] = mf;
  });
  wave_sync();
  local_solve<UT, true>(r, sm, lane / UT, lane % UT, a.rho, a.U);
}

template <int UT, bool QUAD>
__device__ __forceinline__ float pd_backward_task(const BwdArgs &a, int task, BwdLds<UT> &sm) {
  constexpr int NSYS = 64 / UT;
  const int lane = lane_id();
  const int sme = lane / UT, i = lane % UT;
  const size_t HB = (size_t)a.B * a.U;
  const int nvalid = min(NSYS, a.W - task * NSYS);
  auto seg = [&](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
    const size_t w = (size_t)task * NSYS + s;
    Hw = a.H + w * HB;
    yw = a.y + w * a.B;
    r0 = 0;
    r1 = a.B;
  };
  LocalSolve<UT> r;
  round_solve<UT>(a, sm, r, nvalid, seg);
  const bool live = sme < nvalid && i < a.U;
  const size_t w = (size_t)task * NSYS + sme;
  float2 gzc = make_float2(0.f, 0.f);
  float gsc = 0.f;
  if (live) {
    if (a.gz) gzc = a.gz[w * a.U + i];
    if (a.gs) gsc = a.gs[w * a.U + i];
  }
  return round_grads<UT, QUAD>(a, sm, r, nvalid, seg, gzc, gsc);
}

// All clusters of subcarriers w0 .. w0+nsub-1 (nsub = 1 if nw > 1), in rounds
// of NSYS clusters that the nw waves take in turn.  ONCE: each wave has at
// most one round.
template <int UT, bool QUAD, bool ONCE>
__device__ __forceinline__ float fd_backward_task(const BwdArgs &a, int w0, int nsub, BwdLds<UT> *sms, int wv, int nw) {
  constexpr int NSYS = 64 / UT;
  BwdLds<UT> &sm = sms[wv];
  const int lane = lane_id();
  const int sme = lane / UT, i = lane % UT;
  const size_t HB = (size_t)a.B * a.U;
  const int C = a.C, U = a.U;
  const int ntot = nsub * C;
  const bool optimal = a.nu == nullptr;
  // lane groups per subcarrier of a round (C is 1 or 2 when it holds several)
  const int gw = a.spw > 1 ? C : NSYS;
  float gn0 = 0.f;
  LocalSolve<UT> r;
  float S = 0.f, zx = 0.f, zy = 0.f;  // sums over the clusters of the group's subcarrier, user i

  auto make_seg = [&a, C, w0, HB](int base) {
    return [&a, base, C, w0, HB](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
      const int idx = base + s;
      const int wl = idx / C, c = idx - wl * C;
      const size_t w = (size_t)(w0 + wl);
      Hw = a.H + w * HB;
      yw = a.y + w * a.B;
      cluster_rows<BwdArgs>(c, r0, r1);
    };
  };
  auto accumulate = [&](int base) {
    const bool live = base + sme < ntot;
    const float p = live ? 1.0f / (a.n0 * r.d) : 0.f;
    S += group_sum<UT>(p, gw);
    zx += group_sum<UT>(live ? p * r.z.x : 0.f, gw);
    zy += group_sum<UT>(live ? p * r.z.y : 0.f, gw);
  };
  auto meet = [&]() {
    if (nw == 1) return;
    float *part = &sm.M[0][0].x;
    wave_sync();
    if (lane < UT) {
      part[lane] = S;
      part[UT + lane] = zx;
      part[2 * UT + lane] = zy;
    }
    __syncthreads();
    S = zx = zy = 0.f;
    for (int q = 0; q < nw; ++q) {
      const float *o = &sms[q].M[0][0].x;
      S += o[i];
      zx += o[UT + i];
      zy += o[2 * UT + i];
    }
    __syncthreads();
  };
  auto grads = [&](int base) {
    const int nvalid = min(NSYS, ntot - base);
    const int idx = base + sme;
    const int wl = idx / C, c = idx - wl * C;
    const size_t w = (size_t)(w0 + wl);
    float2 gzc = make_float2(0.f, 0.f);
    float gsc = 0.f;
    if (sme < nvalid && i < U) {
      const float2 gz = a.gz ? a.gz[w * U + i] : make_float2(0.f, 0.f);
      const float gs = a.gs ? a.gs[w * U + i] : 0.f;
      const float s2c = a.n0 * r.d;
      float nu;
      if (optimal) {
        const float p = 1.0f / s2c;
        nu = p / S;
        const float gp = (gz.x * (r.z.x - zx / S) + gz.y * (r.z.y - zy / S)) / S;
        gsc = gs * nu * nu - p * p * gp;
      } else {
        nu = a.nu[(w * C + c) * U + i];
        gsc = gs * nu * nu;
        if (a.gnu) a.gnu[(w * C + c) * U + i] = gz.x * r.z.x + gz.y * r.z.y + 2.f * gs * nu * s2c;
      }
      gzc = make_float2(nu * gz.x, nu * gz.y);
    }
    gn0 += round_grads<UT, QUAD>(a, sm, r, nvalid, make_seg(base), gzc, gsc);
  };

  if constexpr (ONCE) {
    const int base = wv * NSYS;
    const bool mine = base < ntot;
    if (mine) {
      round_solve<UT>(a, sm, r, min(NSYS, ntot - base), make_seg(base));
      if (optimal) accumulate(base);
    }
    if (optimal) meet();
    if (mine) grads(base);
  } else {
    if (optimal) {
      for (int base = wv * NSYS; base < ntot; base += nw * NSYS) {
        round_solve<UT>(a, sm, r, min(NSYS, ntot - base), make_seg(base));
        accumulate(base);
        wave_sync();
      }
      meet();
    }
    for (int base = wv * NSYS; base < ntot; base += nw * NSYS) {
      round_solve<UT>(a, sm, r, min(NSYS, ntot - base), make_seg(base));
      grads(base);
    }
  }
  return gn0;
}

// Sum of the workgroup's shares of grad_N0, in wave order.
__device__ __forceinline__ void put_gn0(const BwdArgs &a, float g, float *red, int wv, int nw) {
  g = row16_sum(g);
  g = groups_sum(g);
  if (nw == 1) {
    if (lane_id() == 0) a.gn0_part[blockIdx.x] = g;
    return;
  }
  if (lane_id() == 0) red[wv] = g;
  __syncthreads();
  if (wv == 0 && lane_id() == 0) {
    float s = 0.f;
    for (int q = 0; q < nw; ++q) s += red[q];
    a.gn0_part[blockIdx.x] = s;
  }
}

template <int UT, bool QUAD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(UT == 16 ? 4 : 2, 8))) void eq_backward_pd_kernel(const BwdArgs a) {
  __shared__ BwdLds<UT> sm;
  put_gn0(a, pd_backward_task<UT, QUAD>(a, blockIdx.x, sm), nullptr, 0, 1);
}

// Waves per FD workgroup, at most.
constexpr int kBwdWaves = 8;
template <int UT, bool QUAD, bool ONCE>
__global__ __launch_bounds__(64 * kBwdWaves) __attribute__((amdgpu_waves_per_eu(UT == 16 ? 4 : 2, 8))) void eq_backward_fd_kernel(
    const BwdArgs a) {
  extern __shared__ __align__(128) float2 bwd_lds[];
  BwdLds<UT> *sm = reinterpret_cast<BwdLds<UT> *>(bwd_lds);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), nw = blockDim.x / 64;
  const int w0 = blockIdx.x * a.spw;
  const float g = fd_backward_task<UT, QUAD, ONCE>(a, w0, min(a.spw, a.W - w0), sm, wv, nw);
  if (nw > 1) __syncthreads();
  put_gn0(a, g, reinterpret_cast<float *>(bwd_lds), wv, nw);
}

// Deterministic sum of the per-workgroup shares into the grad_N0 scalar.
__global__ __launch_bounds__(1024) void sum_parts_kernel(const float *__restrict__ part, int n, float *out) {
  __shared__ float red[1024];
  float s = 0.f;
#pragma unroll 8
  for (int t = threadIdx.x; t < n; t += 1024) s += part[t];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 512; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

int backward_tasks(int W, int U, int C, bool fd, int *spw) {
  const int UT = ut_for(U);
  const int nsys = 64 / UT;
  *spw = fd_spw(UT, C);
  return fd ? (W + *spw - 1) / *spw : (W + nsys - 1) / nsys;
}

// Layout of the second pass where gs is zero.  The MFMA layout needs fewer
// instructions, but its lanes take 16 bytes (8 where U is not a multiple of 4)
// of 16 rows at a time, and where the launch fills the chip those accesses
// bound it: then rows of 128 bytes (U = 16) and those of odd lengths above 8
// users take the streaming layout, but for 17 and 18 users, where its second
// half row is nearly empty.  MFMA / streaming, us, PD: 9,600 subcarriers of B =
// 256, U = 7: 138 / 146, U = 8: 127 / 150, U = 12: 180 / 198, U = 15: 276 / 237, U
// = 16: 232 / 213, U = 17: 316 / 317, U = 31: 684 / 422, U = 32: 408 / 425; 1,200 of
// them (300 waves), U = 16: 56 / 76.  60,000 of B = 16, U = 1: 72 / 90.
static bool stream_rows(int U, int waves) {
  return U > 8 && (U % 4 != 0 ? U % 16 > 2 : U == 16) && waves > 512;
}

template <int UT, bool QUAD>
static void launch_bwd(BwdArgs a, bool fd, int ntasks, hipStream_t s) {
  if (!fd) {
    a.stream_rows = stream_rows(a.U, ntasks);
    hipLaunchKernelGGL((eq_backward_pd_kernel<UT, QUAD>), dim3(ntasks), dim3(64), 0, s, a);
    return;
  }
  const int rounds = a.spw > 1 ? 1 : (a.C * UT + 63) / 64;
  const int nw = waves_in_launch(ntasks, rounds < kBwdWaves ? rounds : kBwdWaves);
  a.stream_rows = stream_rows(a.U, ntasks > 512 ? ntasks : ntasks * nw);
  const dim3 grid(ntasks), block(64 * nw);
  const size_t lds = nw * sizeof(BwdLds<UT>);
  if (rounds <= nw)
    hipLaunchKernelGGL((eq_backward_fd_kernel<UT, QUAD, true>), grid, block, lds, s, a);
  else
    hipLaunchKernelGGL((eq_backward_fd_kernel<UT, QUAD, false>), grid, block, lds, s, a);
}

hipError_t launch_backward(const BwdArgs &a, bool fd, int ntasks, hipStream_t s) {
  const bool quad = a.U % 4 == 0;
  if (ut_for(a.U) == 16) {
    if (quad) launch_bwd<16, true>(a, fd, ntasks, s);
    else launch_bwd<16, false>(a, fd, ntasks, s);
  } else {
    if (quad) launch_bwd<32, true>(a, fd, ntasks, s);
    else launch_bwd<32, false>(a, fd, ntasks, s);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.gn0) {
    hipLaunchKernelGGL(sum_parts_kernel, dim3(1), dim3(1024), 0, s, a.gn0_part, ntasks, a.gn0);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace dbpeq
