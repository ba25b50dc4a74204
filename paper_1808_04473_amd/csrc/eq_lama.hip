// LAMA-PD and LAMA-FD (Algorithm 1; Section IV with the normalisation of the
// proof of Lemma 2).  The same fused Gram + matched-filter pass as the
// L-MMSE kernels (G stored unshifted), then every lane group iterates on
// its system's statistics held in registers:
//     z = y^MRC + (I - G) s + v,   tau = N0 + beta phi
//     s' = F(z, tau),   phi' = <G(z, tau)>,   v' = beta phi' / tau (z - s)
// Lane i keeps row i of G (conjugated, so that the DPP-broadcast product
// that forms X^H t in the L-MMSE solve gives (G s)_i here), and s_i, v_i.
// The posterior mean and variance of a square-QAM point factor into those of
// two PAM coordinates (the prior is a product of uniform PAMs and the CN(0,
// tau) likelihood a product of N(0, tau/2) ones).
//
// FD runs the iteration in every cluster on G_c / w_c, y_c^MRC / w_c with
// noise N0 / w_c and system ratio beta / w_c (w_c = B_c / B), then fuses the
// local estimates with Lemma 1's weights built from N0/w_c + (beta/w_c) phi_c.
//
// Up to 16 receive vectors of one channel matrix share the pass over H and the
// row of G, and iterate one after the other.  eq_symbols.hip iterates on all
// vectors of a system at once, on MFMA: better where they are many
// (lama_by_vector).
#include "eq_lama.h"
#include "eq_tiles.h"

namespace dbpeq {

struct LamaOut {
  float2 z;
  float s2;
};

// LDS of one wave: G of the round's systems (swizzled rows, lds_el) and the
// matched filters of its vectors.
template <int UT>
struct LamaLds {
  float2 (*A)[UT][UT];       // [NSYS]
  float2 (*M)[64 / UT][UT];  // [vectors][NSYS]
};
template <int UT>
constexpr size_t lama_lds_bytes(int nv) {
  return (64 / UT) * UT * (UT + nv) * sizeof(float2);
}

// ---------------------------------------------------------------- Gram and the matched filters of NV vectors
// gram_stream with NV receive vectors, vector n of them B entries past the
// first; the vectors from nv on read as zero.  done(s, acc, mf): mf[n] is this
// lane's share of vector n's matched filter.
template <int NV>
struct VecSlot : Slot {
  float2 yn[NV - 1];  // as yl, of the vectors 1 ..
};

template <int UT, int PREC, int NV, class Seg, class Done>
__device__ __forceinline__ void gram_vec_stream(int ns, int U, int B, int nv, Seg seg, Done done) {
  if constexpr (NV == 1) {
    gram_stream<UT, PREC, kLoadLast>(ns, U, seg, [&](int s, const Acc<UT> &acc, float2 mf) {
      const float2 m[1] = {mf};
      done(s, acc, m);
    });
  } else {
    constexpr int RPB = 8 * (64 / UT);
    Acc<UT> acc;
    float2 mf[NV];
    auto zero = [&]() {
      acc_zero<UT>(acc);
#pragma unroll
      for (int n = 0; n < NV; ++n) mf[n] = make_float2(0.f, 0.f);
    };
    zero();
    const LaneOff<UT> lo = lane_offsets<UT>(U);
    SysRef cur;
    int next = 0;
    auto advance = [&]() {
      seg(next, cur.Hw, cur.yw, cur.r0, cur.r1);
      cur.s = next++;
    };
    advance();
    int crb = cur.r0;
    bool more = true;
    auto issue = [&](VecSlot<NV> &sl) -> bool {
      const bool valid = more;
      load_slot<UT, kLoadLast>(sl, lo, cur.Hw, cur.yw, U, crb, cur.r0, cur.r1, valid);
#pragma unroll
      for (int n = 1; n < NV; ++n) {
        const int len = valid && n < nv ? (cur.r1 - cur.r0) * 8 : 0;
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(cur.yw + (size_t)n * B + cur.r0), (short)0, len, kBufFlags);
        sl.yn[n - 1] = buf_ld2<kLoadLast>(ry, lo.y + (unsigned)((crb - cur.r0) * 8));
      }
      sl.s = cur.s;
      sl.last = crb + RPB >= cur.r1;
      if (valid) {
        if (crb + RPB < cur.r1) {
          crb += RPB;
        } else if (next < ns) {
          advance();
          crb = cur.r0;
        } else {
          more = false;
        }
      }
      return valid;
    };
    auto body = [&](const VecSlot<NV> &b) {
      gram_blk<UT, PREC>(b, U, acc, mf[0].x, mf[0].y);
      sfor<NV - 1>([&](auto N) {
        constexpr int n = N;
        sfor<8>([&](auto E) {
          constexpr int e = E;
          fmac_rowbcast<e, false, e == 0 ? 4 : 0>(mf[n + 1].x, b.yn[n].x, b.h[e].x);
          fmac_rowbcast<e, false, 0>(mf[n + 1].y, b.yn[n].y, b.h[e].x);
          fmac_rowbcast<e, false, 0>(mf[n + 1].x, b.yn[n].y, b.h[e].y);
          fmac_rowbcast<e, true, 0>(mf[n + 1].y, b.yn[n].x, b.h[e].y);
        });
      });
    };
    auto fin = [&](const VecSlot<NV> &b) {
      done(b.s, acc, mf);
      zero();
    };
    stream_ring3<VecSlot<NV>>(issue, body, fin);
  }
}

// Vectors per pass of the widest form, whose matched filters come from the
// MFMA tiles: 24 products for 16 vectors against 32 FMACs for each.
constexpr int kLamaTile = 16;

// Streams the round's ns systems into sm; identity systems in the slots past
// them.
template <int UT, int PREC, int NV, bool FD, class Seg>
__device__ __forceinline__ void lama_round(const FwdArgs &a, const LamaLds<UT> &sm, int ns, int nv, Seg seg) {
  const int lane = lane_id();
  if constexpr (NV == kLamaTile) {
    constexpr int NT = UT / 16;
    const int kk = lane / 16, c = lane % 16;
    gram_mf_stream<NT, 1, PREC, sym_rows(NT, FD)>(
        ns, a.U, a.B, nv, seg, [&](int s, const TileAcc<NT> &acc, const TileMf<NT, 1> &m) {
          Tiles<2 * NT - 1> G;
          Tiles<NT> Y;
          tile_gram<NT, PREC>(tile_addr(), lds_addr(sm.A[s]), acc, G);
          tile_mf<NT, PREC>(m, 0, Y);
          wave_sync();
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int u = 4 * kk + r;
              lds_el<UT>(sm.A[s], 16 * t + u, 16 * t + c) = make_float2(G.re[2 * t][r], G.im[2 * t][r]);
              if (NT == 2 && t == 1) {
                lds_el<UT>(sm.A[s], 16 + u, c) = make_float2(G.re[1][r], G.im[1][r]);
                lds_el<UT>(sm.A[s], c, 16 + u) = make_float2(G.re[1][r], -G.im[1][r]);
              }
              if (c < nv) sm.M[c][s][16 * t + u] = make_float2(Y.re[t][r], Y.im[t][r]);
            }
        });
  } else {
    gram_vec_stream<UT, PREC, NV>(ns, a.U, a.B, nv, seg, [&](int s, const Acc<UT> &acc, const float2 (&mf)[NV]) {
      store_gram<UT, PREC>(sm.A[s], acc);
#pragma unroll
      for (int n = 0; n < NV; ++n) {
        const float2 mc = make_float2(colsum<UT>(mf[n].x), colsum<UT>(mf[n].y));
        if (lane < UT) sm.M[n][s][lane] = mc;
      }
    });
  }
  for (int s = ns; s < 64 / UT; ++s) {
    store_identity<UT>(sm.A[s]);
    if (lane < UT)
      for (int n = 0; n < nv; ++n) sm.M[n][s][lane] = make_float2(0.f, 0.f);
  }
  wave_sync();
}

// Row i of the group's G, conjugated and scaled; returns whether the system's
// statistics hold a non-finite entry.  A non-finite y^MRC counts where the
// call has one vector; in the several-vector calls it is left to give NaN for
// its own.
template <int UT>
__device__ __forceinline__ bool lama_load(const LamaLds<UT> &sm, Columns<UT> &f, int slot, int i, float scale, bool one) {
  bool bad = false;
#pragma unroll
  for (int k = 0; k < UT; ++k) {
    const float2 g = lds_el<UT>(sm.A[slot], i, k);
    bad |= !finite2(g);
    f.x[k] = make_float2(g.x * scale, -g.y * scale);
  }
  if (one) bad |= !finite2(sm.M[0][slot][i]);
  return gany<UT>(bad);
}

// Algorithm 1 for vector n of the system in `slot` (lane i: row i of G,
// y^MRC_i), with the statistics scaled by `scale`, noise n0 and system ratio
// beta.
template <int UT, int M>
__device__ __forceinline__ LamaOut lama_local(const LamaLds<UT> &sm, const Columns<UT> &f, int n, int slot, int i, int U,
                                              float scale, float n0, float beta, float es, int t_max) {
  float2 m = sm.M[n][slot][i];
  m = make_float2(m.x * scale, m.y * scale);
  LamaOut o;
  lama_iterate<UT, M>(f, m, i, U, n0, beta, es, t_max, o.z, o.s2);
  return o;
}

// The nv vectors of subcarriers w0 .. w0+nvalid-1.
template <int UT, int PREC, int M, int NV>
__device__ __forceinline__ void lama_pd_task(const FwdArgs &a, int w0, int nvalid, int nv, const LamaLds<UT> &sm) {
  const int lane = lane_id();
  const int g = lane / UT, i = lane % UT;
  const size_t HB = (size_t)a.B * a.U;
  auto seg = [&](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
    const size_t w = (size_t)w0 + s;
    Hw = a.H + w * HB;
    yw = a.y + w * (size_t)a.ysw;
    r0 = 0;
    r1 = a.B;
  };
  lama_round<UT, PREC, NV, false>(a, sm, nvalid, nv, seg);
  const float beta = (float)a.U / (float)a.B;
  const float nanv = __int_as_float(0x7fc00000);
  Columns<UT> f;  // f.x[k] = conj(G_ik)
  const bool bad = lama_load<UT>(sm, f, g, i, 1.0f, !a.lama_sym);
  const bool live = g < nvalid;
  const int w = w0 + g;
  for (int n = 0; n < nv; ++n) {
    const LamaOut o = lama_local<UT, M>(sm, f, n, g, i, a.U, 1.0f, a.n0, beta, a.es, a.lama_t);
    if (live && i < a.U) {
      const size_t at = (size_t)w * a.zsw + (size_t)n * a.U + i;
      a.z[at] = bad ? make_float2(nanv, nanv) : o.z;
      if (a.s2) a.s2[at] = bad ? nanv : o.s2;
    }
  }
  if (live && i == 0 && a.info) a.info[w] = bad ? -1 : 0;
}

// The nv vectors of subcarrier w, all its clusters.
template <int UT, int PREC, int M, int NV>
__device__ __forceinline__ void lama_fd_task(const FwdArgs &a, int w, int nv, const LamaLds<UT> &sm) {
  constexpr int NSYS = 64 / UT;
  const int lane = lane_id();
  const int g = lane / UT, i = lane % UT;
  const size_t HB = (size_t)a.B * a.U;
  const int C = a.C;
  const bool user_nu = a.nu != nullptr;
  const float nanv = __int_as_float(0x7fc00000);
  const float beta = (float)a.U / (float)a.B;
  // fusion sums of user i: weighted estimates, and the weights (optimal) or
  // nu^2 sigma2_c (given weights); group g holds those of the vectors g, g + NSYS ..
  constexpr int NK = (NV + NSYS - 1) / NSYS;
  float tk[NK], zx[NK], zy[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) tk[k] = zx[k] = zy[k] = 0.f;
  for (int base = 0; base < C; base += NSYS) {
    const int nvalid = min(NSYS, C - base);
    auto seg = [&](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
      Hw = a.H + (size_t)w * HB;
      yw = a.y + (size_t)w * a.ysw;
      cluster_rows<FwdArgs>(base + s, r0, r1);
    };
    lama_round<UT, PREC, NV, true>(a, sm, nvalid, nv, seg);
    const int c = base + g;
    const bool live = g < nvalid;
    // w_c of this lane group's cluster (1 for groups past the round)
    const float wc = live ? (float)(a.off[c + 1] - a.off[c]) / (float)a.B : 1.0f;
    const float iw = 1.0f / wc;
    Columns<UT> f;  // f.x[k] = conj(G_ik) / w_c
    const bool bad = lama_load<UT>(sm, f, g, i, iw, !a.lama_sym);
    if (live && i == 0 && a.info) a.info[(size_t)w * C + c] = bad ? -1 : 0;
    float nu = 0.f;
    if (user_nu && live && i < a.U) nu = a.nu[((size_t)w * C + c) * a.U + i];
    for (int v = 0; v < nv; ++v) {
      const LamaOut o = lama_local<UT, M>(sm, f, v, g, i, a.U, iw, a.n0 * iw, beta * iw, a.es, a.lama_t);
      const float p = user_nu ? nu : 1.0f / o.s2;
      float t = user_nu ? p * p * o.s2 : p, x = p * o.z.x, y = p * o.z.y;
      if (bad) t = x = y = nanv;
      if (!live) t = x = y = 0.f;
      t = group_sum<UT>(t, NSYS);
      x = group_sum<UT>(x, NSYS);
      y = group_sum<UT>(y, NSYS);
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        if (v != g + NSYS * k) continue;
        tk[k] += t;
        zx[k] += x;
        zy[k] += y;
      }
    }
    wave_sync();
  }
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int n = g + NSYS * k;
    if (n >= nv || i >= a.U) continue;
    const float inv = 1.0f / tk[k];
    const size_t at = (size_t)w * a.zsw + (size_t)n * a.U + i;
    a.z[at] = user_nu ? make_float2(zx[k], zy[k]) : make_float2(zx[k] * inv, zy[k] * inv);
    if (a.s2) a.s2[at] = user_nu ? tk[k] : inv;
  }
}

// One wave per workgroup: NSYS subcarriers per work item (PD) or one
// subcarrier with all its clusters (FD), at most NV receive vectors.  3 waves
// per SIMD at UT = 16: the row of G, the iterates and the denoiser's level terms
// spill at 4.  UT = 32: 2, and FD no more than 2 even where the registers would
// hold 3: the LDS holds 8 or 9 waves a CU, and with room for a third on each
// SIMD they spread unevenly (2,500 subcarriers of B = 512, U = 20, C = 8: 122 us
// against 103).
template <int UT, int PREC, bool FD, int M, int NV>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(UT == 16 ? 3 : 2, UT == 32 && FD ? 2 : 8))) void eq_lama_kernel(const FwdArgs a) {
  constexpr bool MANY = NV == kLamaTile;
  extern __shared__ __align__(128) float2 lama_lds[];
  __shared__ __align__(128) float2 own[MANY ? 1 : lama_lds_bytes<UT>(NV) / sizeof(float2)];
  float2 *base = MANY ? lama_lds : own;
  const LamaLds<UT> sm = {reinterpret_cast<float2 (*)[UT][UT]>(base),
                          reinterpret_cast<float2 (*)[64 / UT][UT]>(base + (64 / UT) * UT * UT)};
  const int nv = min(NV, a.nsym);
  if constexpr (FD) {
    lama_fd_task<UT, PREC, M, NV>(a, blockIdx.x, nv, sm);
  } else {
    const int w0 = blockIdx.x * a.spw;
    lama_pd_task<UT, PREC, M, NV>(a, w0, min(a.spw, a.W - w0), nv, sm);
  }
}

// PD systems per wave.  Where one each would be a wave or two per SIMD, many
// iterations want one wave with more of its lane groups at work: 1,200
// subcarriers of B = 256, U = 16, 3 vectors of 64-QAM, 40 iterations took 137 us
// with one system each, 88 with two.
static int lama_pd_share(const FwdArgs &a) {
  const bool few = a.W <= kPdItems && a.nsym * a.lama_t > 40;
  return pd_share(a.W, 64 / ut_for(a.U), few ? kPdItems / 2 : kPdItems);
}

// An iteration of a tile takes as long for one vector as for 16, and about
// as long as 12 (10 above 16 users) of one vector in the lane groups of a
// wave, less where lane groups idle (FD with few clusters, small PD batches).
// The streams differ little, but for that of one or two vectors, which needs
// no MFMA for their matched filters.  Tile / vector by vector, us, at 64-QAM.
// FD, 4,800 subcarriers of B = 256, C = 8, U = 16: 1 vector, 10 iterations 581 /
// 80; 4, 1: 52 / 70; 4, 2: 107 / 88; 8, 4: 225 / 212; 10, 10: 583 / 545; 14, 10:
// 584 / 872.  PD, 2,400 of B = 512, U = 32: 2, 3: 113 / 98; 4, 3: 114 / 129; 4,
// 10: 194 / 165; 8, 10: 194 / 217.
bool lama_by_vector(const FwdArgs &a, bool fd) {
  const int n = a.nsym;
  if (n > kLamaTile) return false;
  const int groups = 64 / ut_for(a.U);
  // systems, and the lane groups that the waves of as many rounds hold
  const int sys = fd ? a.C : lama_pd_share(a);
  const int held = (sys + groups - 1) / groups * groups;
  const int most = a.U > 16 ? 10 : 12;
  return n == 1 || n * a.lama_t * held + (n == 2 ? -6 : 4) * sys <= most * (a.lama_t - 1) * sys;
}

template <int UT, int PREC, bool FD, int M, int NV>
static hipError_t launch_lama_one(const FwdArgs &a, hipStream_t s) {
  FwdArgs b = a;
  b.spw = FD ? 1 : lama_pd_share(a);
  hipLaunchKernelGGL((eq_lama_kernel<UT, PREC, FD, M, NV>), dim3((a.W + b.spw - 1) / b.spw), dim3(64),
                     NV == kLamaTile ? lama_lds_bytes<UT>(a.nsym) : 0, s, b);
  return hipGetLastError();
}

template <int UT, int PREC, bool FD, int M>
static hipError_t launch_lama_nv(const FwdArgs &a, hipStream_t s) {
  // the narrowest form that holds the vectors
  if (a.nsym == 1) return launch_lama_one<UT, PREC, FD, M, 1>(a, s);
  if (a.nsym == 2) return launch_lama_one<UT, PREC, FD, M, 2>(a, s);
  if constexpr (UT == 16)
    if (a.nsym <= 4) return launch_lama_one<UT, PREC, FD, M, 4>(a, s);
  return launch_lama_one<UT, PREC, FD, M, kLamaTile>(a, s);
}

template <int UT, int PREC, bool FD>
static hipError_t launch_lama_m(const FwdArgs &a, hipStream_t s) {
  switch (a.lama_m) {
    case 2: return launch_lama_nv<UT, PREC, FD, 2>(a, s);
    case 4: return launch_lama_nv<UT, PREC, FD, 4>(a, s);
    case 8: return launch_lama_nv<UT, PREC, FD, 8>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int UT, bool FD>
static hipError_t launch_lama_prec(const FwdArgs &a, int prec, hipStream_t s) {
  return prec == PREC_FP32 ? launch_lama_m<UT, PREC_FP32, FD>(a, s) : launch_lama_m<UT, PREC_BF16X3_NR, FD>(a, s);
}

hipError_t launch_lama(const FwdArgs &a, bool fd, int prec, hipStream_t s) {
  if (prec != PREC_FP32 && prec != PREC_BF16X3_NR) return hipErrorInvalidValue;
  if (a.nsym < 1 || a.nsym > kLamaTile) return hipErrorInvalidValue;
  const int UT = ut_for(a.U);
  if (UT == 16) return fd ? launch_lama_prec<16, true>(a, prec, s) : launch_lama_prec<16, false>(a, prec, s);
  return fd ? launch_lama_prec<32, true>(a, prec, s) : launch_lama_prec<32, false>(a, prec, s);
}

}  // namespace dbpeq
