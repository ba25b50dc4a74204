// Several receive vectors per channel matrix (Section VI-B).
//
// The OFDM symbols of one coherence interval share the channel, so the Gram
// matrix of a subcarrier (PD) or cluster (FD) and its factor are formed once
// and applied to every symbol; only the matched filter is formed per symbol.
// The matched filters of up to 16 symbols (PD with more than 16 users: 32),
// H_c^H [y_1 .. y_S], are a second MFMA product in the same pass over H, and H
// and the receive vectors are each read from HBM once per launch.
//
// The streams, in 16 x 16 tiles, are those of eq_tiles.h.  A result in MFMA
// accumulator layout is the B operand of a next product whose k index runs as
// (register, lane group), so matched filters and estimates go from product to
// product in registers.
//
// L-MMSE / ZF: each lane group factors its system (solve_slot) and leaves X =
// L^{-1} in LDS; the estimates of all symbols are Z = X^H (X M), two products
// per system.  MRC and LAMA (Algorithm 1) need no factor and work on one
// system at a time as its stream ends, for all symbols at once.
//
// FD weights every cluster's estimates with the weights of Lemma 1 (or given
// ones) and sums them over the clusters: each wave of the workgroup takes a
// share of them in cluster order, and the waves' sums are added in order.
//
// Forms: FP32 MFMA and split-BF16 MFMA (three products per real product)
// without refinement.  Ill-conditioned systems go to the FP64 re-solve queue
// as in the single-vector kernels; the re-solve recomputes every symbol of
// the tile.
#include "eq_lama.h"
#include "eq_tiles.h"

namespace dbpeq {

// Symbol tiles per launch.  PD at 32 users reads H once for 32 symbols: two
// launches of 16 each took 15-25% longer (MRC of 24 vectors, 1,200 subcarriers
// of B = 1024: 228 against 185 us).  The solves bound FD, where a second
// symbol tile in LDS would cost half the waves (two launches for 17 to 32
// vectors take 0.4 to 0.75 of the time of the former one launch).
constexpr int sym_tiles(int UT, bool fd) { return UT == 32 && !fd ? 2 : 1; }

// ---------------------------------------------------------------- outputs
// FD sums in accumulator layout: weighted estimates, and weights (optimal:
// the fused variance is 1 / tk) or nu^2 sigma2_c (given weights: the fused
// variance itself).
template <int NT>
struct FuseSum {
  Tiles<NT> z;
  f4 tk[NT];
};

template <int NT>
__device__ __forceinline__ void fuse_zero(FuseSum<NT> &f) {
  const f4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < NT; ++t) f.z.re[t] = f.z.im[t] = f.tk[t] = z;
}

// Adds the waves' sums in wave order; part(q) is 12 NT * 64 floats of LDS of
// wave q.  Returns true in the wave that holds the result.
template <int NT, int NW, class Part>
__device__ __forceinline__ bool fuse_waves(FuseSum<NT> &f, int wv, Part part) {
  if constexpr (NW == 1) {
    return true;
  } else {
    const int lane = lane_id();
    float *o = part(wv);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        o[(12 * t + r) * 64 + lane] = f.z.re[t][r];
        o[(12 * t + 4 + r) * 64 + lane] = f.z.im[t][r];
        o[(12 * t + 8 + r) * 64 + lane] = f.tk[t][r];
      }
    __syncthreads();
    if (wv != 0) return false;
    fuse_zero<NT>(f);
    for (int q = 0; q < NW; ++q) {
      const float *p = part(q);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          f.z.re[t][r] += p[(12 * t + r) * 64 + lane];
          f.z.im[t][r] += p[(12 * t + 4 + r) * 64 + lane];
          f.tk[t][r] += p[(12 * t + 8 + r) * 64 + lane];
        }
    }
    return true;
  }
}

// Writes the fused estimates of subcarrier w, and sigma2 as [W][U] or (PERSYM)
// [W][S][U].
template <int NT, bool PERSYM>
__device__ __forceinline__ void fuse_write(const FwdArgs &a, int w, const FuseSum<NT> &f) {
  const int lane = lane_id();
  const int kk = lane / 16, c = lane % 16;
  const bool user_nu = a.nu != nullptr;
  const size_t ob = (size_t)w * a.zsw + (size_t)c * a.U;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = 16 * t + 4 * kk + r;
      const float inv = 1.0f / f.tk[t][r];
      const float s = user_nu ? f.tk[t][r] : inv;
      if (u < a.U) {
        if (c < a.nsym) {
          a.z[ob + u] = user_nu ? make_float2(f.z.re[t][r], f.z.im[t][r])
                                : make_float2(f.z.re[t][r] * inv, f.z.im[t][r] * inv);
          if (PERSYM && a.s2) a.s2[ob + u] = s;
        }
        if (!PERSYM && c == 0 && a.s2) a.s2[(size_t)w * a.U + u] = s;
      }
    }
}

__device__ __forceinline__ void enqueue_fp64_sym(const FwdArgs &a, int w) {
  if (!a.fb_count) return;
  const int pos = atomicAdd(a.fb_count, 1);
  if (pos >= 0 && pos < a.W) a.fb_list[pos] = w;  // capacity W
}

// ---------------------------------------------------------------- L-MMSE, ZF
// LDS of one wave: packed matrix slots, and at 32 users the matched filters
// (accumulator layout, one 16-byte word per lane and tile part).  At 16 users
// the matched filters of the round's four systems stay in 32 registers: 8 KB
// of LDS instead of 16 (LDS comes in units of 1,280 bytes: 9 waves per CU).
template <int NT, int NSLOT, int NC = 1>
struct SymLds {
  static constexpr int NS = NSLOT;
  alignas(128) float2 A[NS * kSlot<32>];  // TileAddr flips address bits below 128
  f4 M[NS][NC][4][64];
};
template <int NSLOT>
struct SymLds<1, NSLOT, 1> {
  static constexpr int NS = NSLOT;
  alignas(128) float2 A[NS * kSlot<16>];
};

// Matched filters of the systems of a round.
template <int NT, int NS>
struct SymMf {
  Tiles<1> m[NT == 1 ? NS : 1];
};

template <int NT, int NC, int PREC, class SM>
__device__ __forceinline__ void store_system(SM &sm, const TileAddr &ta, SymMf<NT, SM::NS> &mf, int s, const TileAcc<NT> &acc,
                                             const TileMf<NT, NC> &m) {
  const int lane = lane_id();
  const uint32_t slot = lds_addr(sm.A) + s * (8 * kSlot<16 * NT>);
  Tiles<2 * NT - 1> G;
  tile_gram<NT, PREC>(ta, slot, acc, G);
  wave_sync();
  const uint32_t p = slot + ta.p;
  sfor<2 * NT - 1>([&](auto Bk) {
    constexpr int b = Bk;
    sfor<4>([&](auto R) {
      constexpr int r = R;
      lds_put((p ^ (8 * r)) + 2048 * b + 128 * r, G.re[b][r], G.im[b][r]);
    });
  });
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    Tiles<NT> M;
    tile_mf<NT, PREC>(m, n, M);
    if constexpr (NT == 1) {
      sfor<SM::NS>([&](auto Q) {
        if (s == Q) mf.m[Q] = M;
      });
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        sm.M[s][n][2 * t][lane] = M.re[t];
        sm.M[s][n][2 * t + 1][lane] = M.im[t];
      }
    }
  }
}

// out += X M (HERM = false) or X^H M (HERM = true) for one 16 x 16 block of X,
// whose conjugate the slot holds transposed (row u: column u).  16 users take
// three real products (Gauss), 32 users four: the Gauss form is 25% fewer
// MFMAs of a product that is a tenth of the work there, and rounds more.
template <bool HERM, bool GAUSS>
__device__ __forceinline__ void block_mul(float2 *As, int b, const f4 &mr, const f4 &mi, f4 &k1, f4 &k2, f4 &k3) {
  const int lane = lane_id();
  const int kk = lane / 16, c = lane % 16;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    // A operand [i = c][k = (r, kk)]: X[c][4 kk + r], or conj(X[4 kk + r][c])
    const float2 x = HERM ? blk_el(As, b, c, 4 * kk + r) : blk_el(As, b, 4 * kk + r, c);
    if constexpr (GAUSS) {
      // xr = x.x, xi = +-x.y: k1 = (xr + xi) mr, k2 = xr (mi - mr), k3 = xi (mr + mi);
      // Re = k1 - k3, Im = k1 + k2
      const float xi = HERM ? x.y : -x.y;
      k1 = mma32(x.x + xi, mr[r], k1);
      k2 = mma32(x.x, mi[r] - mr[r], k2);
      k3 = mma32(xi, mr[r] + mi[r], k3);
    } else {
      // k1 = Re, k2 = Im
      k1 = mma32(x.x, mr[r], k1);
      k2 = mma32(x.x, mi[r], k2);
      k1 = mma32(HERM ? -x.y : x.y, mi[r], k1);
      k2 = mma32(HERM ? x.y : -x.y, mr[r], k2);
    }
  }
}

// Z = X^H (X M) for slot q and every symbol of tile n, the whole wave on one
// system.
template <int NT, class SM>
__device__ __forceinline__ void sym_apply(SM &sm, const Tiles<1> &m0, int q, int n, Tiles<NT> &Z) {
  constexpr bool GAUSS = NT == 1;
  const int lane = lane_id();
  float2 *As = sm.A + q * kSlot<16 * NT>;
  const f4 z0 = {0.f, 0.f, 0.f, 0.f};
  Tiles<NT> T;
  f4 mr[NT], mi[NT], k1, k2, k3;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if constexpr (NT == 1) {
      mr[t] = m0.re[0];
      mi[t] = m0.im[0];
    } else {
      mr[t] = sm.M[q][n][2 * t][lane];
      mi[t] = sm.M[q][n][2 * t + 1][lane];
    }
  }
  auto out = [&](f4 &re, f4 &im) {
    re = GAUSS ? k1 - k3 : k1;
    im = GAUSS ? k1 + k2 : k2;
  };
  // T: rows of X (blocks 0; 1, 2)
  k1 = k2 = k3 = z0;
  block_mul<false, GAUSS>(As, 0, mr[0], mi[0], k1, k2, k3);
  out(T.re[0], T.im[0]);
  if constexpr (NT == 2) {
    k1 = k2 = k3 = z0;
    block_mul<false, GAUSS>(As, 1, mr[0], mi[0], k1, k2, k3);
    block_mul<false, GAUSS>(As, 2, mr[1], mi[1], k1, k2, k3);
    out(T.re[1], T.im[1]);
  }
  // Z: columns of X (blocks 0, 1; 2)
  k1 = k2 = k3 = z0;
  block_mul<true, GAUSS>(As, 0, T.re[0], T.im[0], k1, k2, k3);
  if constexpr (NT == 2) block_mul<true, GAUSS>(As, 1, T.re[1], T.im[1], k1, k2, k3);
  out(Z.re[0], Z.im[0]);
  if constexpr (NT == 2) {
    k1 = k2 = k3 = z0;
    block_mul<true, GAUSS>(As, 2, T.re[1], T.im[1], k1, k2, k3);
    out(Z.re[1], Z.im[1]);
  }
}

// Value v of lane group q's user 16 t + 4 kk + r, in accumulator layout.
template <int NT>
__device__ __forceinline__ void to_tiles(float v, int q, f4 (&o)[NT]) {
  const int kk = lane_id() / 16;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) o[t][r] = __shfl(v, q * 16 * NT + 16 * t + 4 * kk + r);
}

// PD: systems w0 .. w0+nvalid-1, one per lane group.
template <int NT, int NC, int PREC, class SM>
__device__ __forceinline__ void pd_sym_task(const FwdArgs &a, int w0, int nvalid, SM &sm) {
  constexpr int UT = 16 * NT;
  const int lane = lane_id();
  const int g = lane / UT, i = lane % UT;
  SymMf<NT, SM::NS> mf;
  const TileAddr ta = tile_addr();
  gram_mf_stream<NT, NC, PREC, sym_rows(NT, false)>(nvalid, a.U, a.B, a.nsym, pd_seg(a, w0), [&](int s, const TileAcc<NT> &acc, const TileMf<NT, NC> &m) {
    store_system<NT, NC, PREC>(sm, ta, mf, s, acc, m);
  });
  wave_sync();
  LocalSolve<UT> r;
  solve_slot<UT, true, SM::NS, false>(r, sm.A, slot_of<SM>(g), i, make_float2(0.f, 0.f), a.rho, a.U);
  wave_sync();
  const bool live = g < nvalid;
  const float kappa = r.norm1 * gsum<UT>(i < a.U ? r.d : 0.f);
  const bool routed = live && !r.bad && (r.fail != 0 || !(kappa <= EQ_COND_LIMIT));
  const int w = w0 + g;
  const float nanv = __int_as_float(0x7fc00000);
  // gain factor of user i (1 unless the unbiased L-MMSE)
  const float ku = a.ub != 0.f ? unbias_factor(a.n0 * r.d, a.ub) : 1.f;
  const float kz = r.bad ? nanv : ku;
  const int kk = lane / 16, c = lane % 16;
  sfor<SM::NS>([&](auto Q) {
    constexpr int q = Q;
    if (q >= nvalid) return;
    f4 k[NT];
    to_tiles<NT>(kz, q, k);
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      Tiles<NT> Z;
      sym_apply<NT>(sm, mf.m[NT == 1 ? q : 0], q, n, Z);
      float2 *zw = a.z + (size_t)(w0 + q) * a.zsw + (size_t)(16 * n + c) * a.U;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int u = 16 * t + 4 * kk + rr;
          if (16 * n + c < a.nsym && u < a.U) zw[u] = make_float2(Z.re[t][rr] * k[t][rr], Z.im[t][rr] * k[t][rr]);
        }
    }
  });
  if (live) {
    if (i < a.U && a.s2) a.s2[(size_t)w * a.U + i] = r.bad ? nanv : a.n0 * r.d * ku;
    if (i == 0) {
      if (a.info) a.info[w] = (r.bad ? -1 : r.fail) | (routed ? EQ_INFO_FP64 : 0);
      if (routed) enqueue_fp64_sym(a, w);
    }
  }
}

// FD: all clusters of subcarrier w, in rounds of NSYS that the NW waves take
// in turn.
template <int NT, int PREC, int NW, class SM>
__device__ __forceinline__ void fd_sym_task(const FwdArgs &a, int w, SM *sms, int wv) {
  constexpr int UT = 16 * NT, NSYS = 64 / UT;
  SM &sm = sms[wv];
  const int lane = lane_id();
  const int C = a.C;
  const bool user_nu = a.nu != nullptr;
  const float nanv = __int_as_float(0x7fc00000);
  FuseSum<NT> f;
  fuse_zero<NT>(f);
  float tk = 0.f;  // the weights' sum of user i, clusters of this lane's group
  bool any = false;
  const int g = lane / UT, i = lane % UT;
  const TileAddr ta = tile_addr();
  for (int base = wv * NSYS; base < C; base += NW * NSYS) {
    const int nvalid = min(NSYS, C - base);
    SymMf<NT, SM::NS> mf;
    gram_mf_stream<NT, 1, PREC, sym_rows(NT, true)>(nvalid, a.U, a.B, a.nsym, fd_seg(a, w, [base](int s) { return base + s; }),
                             [&](int s, const TileAcc<NT> &acc, const TileMf<NT, 1> &m) { store_system<NT, 1, PREC>(sm, ta, mf, s, acc, m); });
    wave_sync();
    LocalSolve<UT> r;
    solve_slot<UT, true, SM::NS, false>(r, sm.A, g, i, make_float2(0.f, 0.f), a.rho, a.U);
    wave_sync();
    const int c = base + g;
    const bool live = g < nvalid;
    const float kappa = r.norm1 * gsum<UT>(i < a.U ? r.d : 0.f);
    const bool routed = live && !r.bad && (r.fail != 0 || !(kappa <= EQ_COND_LIMIT));
    if (live && i == 0 && a.info) a.info[(size_t)w * C + c] = (r.bad ? -1 : r.fail) | (routed ? EQ_INFO_FP64 : 0);
    any |= __ballot(routed) != 0ull;
    // local variance (of the estimate scaled to unit gain for the unbiased
    // L-MMSE: estimate and variance times ku) and fusion weight p; the
    // estimate's weight is p ku
    const float ku = a.ub != 0.f ? unbias_factor(a.n0 * r.d, a.ub) : 1.f;
    const float s2c = a.n0 * r.d * ku;
    float p = 0.f;
    if (live && i < a.U) p = user_nu ? a.nu[((size_t)w * C + c) * a.U + i] : 1.0f / s2c;
    if (live) tk += r.bad ? nanv : (user_nu ? p * p * s2c : p);
    const float pz = r.bad ? nanv : p * ku;
    sfor<SM::NS>([&](auto Q) {
      constexpr int q = Q;
      if (q >= nvalid) return;
      Tiles<NT> Z;
      sym_apply<NT>(sm, mf.m[NT == 1 ? q : 0], q, 0, Z);
      f4 wq[NT];
      to_tiles<NT>(pz, q, wq);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        f.z.re[t] += wq[t] * Z.re[t];
        f.z.im[t] += wq[t] * Z.im[t];
      }
    });
    wave_sync();
  }
  tk = UT == 16 ? groups_sum(tk) : xor32_sum(tk);
  to_tiles<NT>(tk, 0, f.tk);
  if (NW > 1 && lane == 0) sm.A[0].x = any ? 1.f : 0.f;
  if (!fuse_waves<NT, NW>(f, wv, [&](int q) { return (float *)sms[q].A + 64; })) return;
  fuse_write<NT, false>(a, w, f);
  if (NW > 1)
    for (int q = 0; q < NW; ++q) any |= sms[q].A[0].x != 0.f;
  if (lane == 0 && any) enqueue_fp64_sym(a, w);
}

// ---------------------------------------------------------------- MRC (Section III-A)
// 1 / G_uu and sigma2_u = N0 / G_uu + E_s sum_{k != u} |G_uk|^2 / G_uu^2 in
// accumulator layout (equal in every column); fail = u + 1 for the first user
// with G_uu <= 0.
template <int NT>
struct TileMrc {
  f4 inv[NT], s2[NT];
  int fail;
  bool bad;
};

template <int N>
__device__ __forceinline__ bool tiles_bad(const Tiles<N> &G) {
  bool bad = false;
#pragma unroll
  for (int b = 0; b < N; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) bad |= !isfinite(G.re[b][r]) || !isfinite(G.im[b][r]);
  return __ballot(bad) != 0ull;
}

template <int NT>
__device__ __forceinline__ TileMrc<NT> tile_mrc(const Tiles<2 * NT - 1> &G, int U, float n0, float es) {
  const int lane = lane_id();
  const int kk = lane / 16, c = lane % 16;
  TileMrc<NT> o;
  o.bad = tiles_bad<2 * NT - 1>(G);
  float below = 0.f;  // NT = 2: sum_k |G_{16 + k, c}|^2, user c of the first tile
  if constexpr (NT == 2) {
#pragma unroll
    for (int r = 0; r < 4; ++r) below = fmaf(G.re[1][r], G.re[1][r], fmaf(G.im[1][r], G.im[1][r], below));
    below = groups_sum(below);
  }
  int fail = 4 * EQ_MAX_U;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = 16 * t + 4 * kk + r;
      const float re = G.re[2 * t][r], im = G.im[2 * t][r];
      const bool diag = c == 4 * kk + r;
      float off = diag ? 0.f : fmaf(re, re, im * im);
      if (NT == 2 && t == 1) off = fmaf(G.re[1][r], G.re[1][r], fmaf(G.im[1][r], G.im[1][r], off));
      off = row16_sum(off);
      if (NT == 2 && t == 0) off += __shfl(below, 4 * kk + r);
      const float gii = row16_sum(diag ? re : 0.f);
      if (u < U && !(gii > 0.f)) fail = min(fail, u + 1);
      const float inv = 1.0f / gii;
      o.inv[t][r] = inv;
      o.s2[t][r] = n0 * inv + es * off * inv * inv;
    }
  fail = min(fail, __shfl_xor(fail, 16));
  fail = min(fail, __shfl_xor(fail, 32));
  o.fail = fail <= EQ_MAX_U ? fail : 0;
  return o;
}

// ---------------------------------------------------------------- LAMA (Algorithm 1)
// t_max iterations for one system and every symbol of the tile:
//     z = y^MRC + (I - G) s + v,   tau = N0 + beta phi,
//     s' = F(z, tau),   phi' = <G(z, tau)>,   v' = beta phi' / tau (z - s),
// G s on MFMA (the Gram registers are their own A operand: lane (kk, c) holds
// G_{4 kk + r, c} = conj(G_{c, 4 kk + r})), the rest per element.  The first
// iteration has s = v = 0, so z = y^MRC; the last one ends with z and tau.
// Returns z in Z and the symbol's variance N0 + beta phi.
template <int NT, int M>
__device__ __forceinline__ float tile_lama(const Tiles<2 * NT - 1> &G, const Tiles<1> &G01t, const Tiles<NT> &Y, int U,
                                           float n0, float beta, float es, int t_max, Tiles<NT> &Z) {
  const int kk = lane_id() / 16;
  const float lvl = sqrtf(3.0f * es / (2.0f * (float)(M * M - 1)));
  const float inv_u = 1.0f / (float)U;
  Tiles<NT> S, V;
  Z = Y;
  float tau = n0 + beta * es;
  for (int it = 1; it < t_max; ++it) {
    // posterior of the previous z
    const float inv_tau = 1.0f / tau;
    float g = 0.f;
    Tiles<NT> N;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float mr, qr, mi, qi;
        pam_posterior<M>(Z.re[t][r], inv_tau, lvl, mr, qr);
        pam_posterior<M>(Z.im[t][r], inv_tau, lvl, mi, qi);
        const bool user = 16 * t + 4 * kk + r < U;
        N.re[t][r] = user ? mr : 0.f;
        N.im[t][r] = user ? mi : 0.f;
        g += user ? (qr - mr * mr) + (qi - mi * mi) : 0.f;
      }
    const float phi = groups_sum(g) * inv_u;
    const float k = beta * phi * inv_tau;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (it == 1) {
        V.re[t] = k * Z.re[t];
        V.im[t] = k * Z.im[t];
      } else {
        V.re[t] = k * (Z.re[t] - S.re[t]);
        V.im[t] = k * (Z.im[t] - S.im[t]);
      }
    }
    S = N;
    tau = n0 + beta * phi;
    // z = y^MRC + s - G s + v
    Tiles<NT> P;
    const f4 z0 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f4 pr = z0, pi = z0;
#pragma unroll
      for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // G_{16 t + c, 16 b + 4 kk + r}
          const bool low = NT == 2 && t == 1 && b == 0;
          const int blk = t == b ? 2 * t : 1;
          const float gr = low ? G01t.re[0][r] : G.re[blk][r];
          const float gi = low ? G01t.im[0][r] : -G.im[blk][r];
          pr = mma32(gr, S.re[b][r], pr);
          pi = mma32(gr, S.im[b][r], pi);
          pr = mma32(-gi, S.im[b][r], pr);
          pi = mma32(gi, S.re[b][r], pi);
        }
      P.re[t] = pr;
      P.im[t] = pi;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      Z.re[t] = Y.re[t] + S.re[t] - P.re[t] + V.re[t];
      Z.im[t] = Y.im[t] + S.im[t] - P.im[t] + V.im[t];
    }
  }
  return tau;
}

// NT = 2: block (1, 0) with rows and columns exchanged, G_{16 + c, 4 kk + r} at
// lane (kk, c), through 512 floats of LDS.
template <int NT>
__device__ __forceinline__ void tile_turn(float *scratch, const Tiles<2 * NT - 1> &G, Tiles<1> &o) {
  if constexpr (NT == 2) {
    const int lane = lane_id();
    const int kk = lane / 16, c = lane % 16;
    wave_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = 4 * kk + r;
      scratch[16 * u + (c ^ u)] = G.re[1][r];
      scratch[256 + 16 * u + (c ^ u)] = G.im[1][r];
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = 4 * kk + r;
      o.re[0][r] = scratch[16 * c + (u ^ c)];
      o.im[0][r] = scratch[256 + 16 * c + (u ^ c)];
    }
  }
}

// ---------------------------------------------------------------- MRC and LAMA kernels
// M = 0: MRC; else LAMA with M levels per coordinate.  LDS of one wave: the
// transposes' scratch and, at the end, the wave's fusion sums.
template <int NT>
struct DirectLds {
  alignas(128) float f[12 * NT * 64];
};

// One system (PD): estimates and variances to their rows.
template <int NT, int NC, int PREC, int M>
__device__ __forceinline__ void pd_direct_task(const FwdArgs &a, int w0, int nvalid, DirectLds<NT> &sm) {
  const int lane = lane_id();
  const int kk = lane / 16, c = lane % 16;
  const float nanv = __int_as_float(0x7fc00000);
  gram_mf_stream<NT, NC, PREC, sym_rows(NT, false)>(nvalid, a.U, a.B, a.nsym, pd_seg(a, w0), [&](int s, const TileAcc<NT> &acc, const TileMf<NT, NC> &m) {
    const int w = w0 + s;
    Tiles<2 * NT - 1> G;
    tile_gram<NT, PREC>(tile_addr(), lds_addr(sm.f), acc, G);
    TileMrc<NT> o;
    Tiles<1> T;
    int code;
    if constexpr (M == 0) {
      o = tile_mrc<NT>(G, a.U, a.n0, a.es);
      code = o.bad ? -1 : o.fail;
    } else {
      tile_turn<NT>(sm.f, G, T);
      code = tiles_bad<2 * NT - 1>(G) ? -1 : 0;
    }
    const bool out_nan = code != 0;
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      Tiles<NT> Y, Z;
      tile_mf<NT, PREC>(m, n, Y);
      f4 s2[NT];
      if constexpr (M == 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          Z.re[t] = Y.re[t] * o.inv[t];
          Z.im[t] = Y.im[t] * o.inv[t];
          s2[t] = o.s2[t];
        }
      } else {
        const float tau = tile_lama<NT, M>(G, T, Y, a.U, a.n0, (float)a.U / (float)a.B, a.es, a.lama_t, Z);
#pragma unroll
        for (int t = 0; t < NT; ++t) s2[t] = tau;
      }
      const int sym = 16 * n + c;
      const size_t ob = (size_t)w * a.zsw + (size_t)sym * a.U;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int u = 16 * t + 4 * kk + r;
          if (u < a.U) {
            const float v = out_nan ? nanv : s2[t][r];
            if (sym < a.nsym) {
              a.z[ob + u] = out_nan ? make_float2(nanv, nanv) : make_float2(Z.re[t][r], Z.im[t][r]);
              if (M != 0 && a.s2) a.s2[ob + u] = v;
            }
            if (M == 0 && sym == 0 && a.s2) a.s2[(size_t)w * a.U + u] = v;
          }
        }
    }
    if (lane == 0 && a.info) a.info[w] = code;
  });
}

// All clusters of subcarrier w, shared among the NW waves.  LAMA-FD runs on
// the statistics normalised by 1 / w_c, w_c = B_c / B.
template <int NT, int PREC, int M, int NW>
__device__ __forceinline__ void fd_direct_task(const FwdArgs &a, int w, DirectLds<NT> *sms, int wv) {
  DirectLds<NT> &sm = sms[wv];
  const int lane = lane_id();
  const int kk = lane / 16;
  const bool user_nu = a.nu != nullptr;
  const float nanv = __int_as_float(0x7fc00000);
  const int C = a.C;
  FuseSum<NT> f;
  fuse_zero<NT>(f);
  const int ncl = wv < C ? (C - wv + NW - 1) / NW : 0;
  auto cluster = [wv](int s) { return wv + NW * s; };
  if (ncl > 0)
    gram_mf_stream<NT, 1, PREC, sym_rows(NT, true)>(ncl, a.U, a.B, a.nsym, fd_seg(a, w, cluster), [&](int s, const TileAcc<NT> &acc, const TileMf<NT, 1> &m) {
      const int c = cluster(s);
      Tiles<2 * NT - 1> G;
      Tiles<NT> Y, Z;
      tile_gram<NT, PREC>(tile_addr(), lds_addr(sm.f), acc, G);
      tile_mf<NT, PREC>(m, 0, Y);
      f4 s2[NT];
      int code;
      if constexpr (M == 0) {
        const TileMrc<NT> o = tile_mrc<NT>(G, a.U, a.n0, a.es);
        code = o.bad ? -1 : o.fail;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          Z.re[t] = Y.re[t] * o.inv[t];
          Z.im[t] = Y.im[t] * o.inv[t];
          s2[t] = o.s2[t];
        }
      } else {
        int r0, r1;
        cluster_rows<FwdArgs>(c, r0, r1);
        const float iw = 1.0f / ((float)(r1 - r0) / (float)a.B);
        code = tiles_bad<2 * NT - 1>(G) ? -1 : 0;  // of G itself: 1 / w_c may overflow it
#pragma unroll
        for (int b = 0; b < 2 * NT - 1; ++b) {
          G.re[b] *= iw;
          G.im[b] *= iw;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          Y.re[t] *= iw;
          Y.im[t] *= iw;
        }
        Tiles<1> T;
        tile_turn<NT>(sm.f, G, T);
        const float tau = tile_lama<NT, M>(G, T, Y, a.U, a.n0 * iw, (float)a.U / (float)a.B * iw, a.es, a.lama_t, Z);
#pragma unroll
        for (int t = 0; t < NT; ++t) s2[t] = tau;
      }
      if (lane == 0 && a.info) a.info[(size_t)w * C + c] = code;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int u = 16 * t + 4 * kk + r;
          float p = 0.f;
          if (u < a.U) p = user_nu ? a.nu[((size_t)w * C + c) * a.U + u] : 1.0f / s2[t][r];
          if (code != 0) p = nanv;
          f.z.re[t][r] += p * Z.re[t][r];
          f.z.im[t][r] += p * Z.im[t][r];
          f.tk[t][r] += user_nu ? p * p * s2[t][r] : p;
        }
    });
  if (!fuse_waves<NT, NW>(f, wv, [&](int q) { return sms[q].f; })) return;
  fuse_write<NT, M != 0>(a, w, f);
}

// ---------------------------------------------------------------- kernels
// Most PD systems per work item: a round of lane groups.
template <int NT>
constexpr int sym_pd_per() {
  return NT == 1 ? 4 : 1;
}

// The launch arguments of block row y of the grid: its 16 vectors.  The others
// of a subcarrier leave what does not depend on the vector to row 0.
template <bool PERSYM>
__device__ __forceinline__ FwdArgs tile_args(const FwdArgs &a) {
  FwdArgs b = a;
  const int s0 = 16 * blockIdx.y;
  b.nsym = min(16, a.nsym - s0);
  b.y += (size_t)s0 * a.B;
  b.z += (size_t)s0 * a.U;
  if (PERSYM && a.s2) b.s2 += (size_t)s0 * a.U;
  if (s0) {
    if (!PERSYM) b.s2 = nullptr;
    b.info = nullptr;
    b.fb_count = nullptr;
  }
  return b;
}

template <int NT, int NC, int PREC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NT == 1 ? 3 : 2, 8))) void eq_symbols_pd_kernel(const FwdArgs a) {
  __shared__ SymLds<NT, sym_pd_per<NT>(), NC> sm;
  const int w0 = blockIdx.x * a.spw;
  if constexpr (NT == 2 && NC == 1)
    pd_sym_task<NT, NC, PREC>(tile_args<false>(a), w0, min(a.spw, a.W - w0), sm);
  else
    pd_sym_task<NT, NC, PREC>(a, w0, min(a.spw, a.W - w0), sm);
}

template <int NT, int PREC, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NT == 1 && PREC == PREC_FP32 ? 4 : NT == 1 ? 3 : 2, 8))) void eq_symbols_fd_kernel(const FwdArgs a) {
  __shared__ SymLds<NT, 4 / NT> sm[NW];
  fd_sym_task<NT, PREC, NW>(a, blockIdx.x, sm, __builtin_amdgcn_readfirstlane(threadIdx.x / 64));
}

template <int NT, int NC, int PREC, int M>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8))) void eq_direct_pd_kernel(const FwdArgs a) {
  __shared__ DirectLds<NT> sm;
  const int w0 = blockIdx.x * a.spw;
  if constexpr (NT == 2 && NC == 1)
    pd_direct_task<NT, NC, PREC, M>(tile_args<M != 0>(a), w0, min(a.spw, a.W - w0), sm);
  else
    pd_direct_task<NT, NC, PREC, M>(a, w0, min(a.spw, a.W - w0), sm);
}

template <int NT, int PREC, int M, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 8))) void eq_direct_fd_kernel(const FwdArgs a) {
  __shared__ DirectLds<NT> sm[NW];
  fd_direct_task<NT, PREC, M, NW>(a, blockIdx.x, sm, __builtin_amdgcn_readfirstlane(threadIdx.x / 64));
}

template <int NT, int PREC, int NW>
static void launch_fd(const FwdArgs &a, hipStream_t s) {
  hipLaunchKernelGGL((eq_symbols_fd_kernel<NT, PREC, NW>), dim3(a.W), dim3(64 * NW), 0, s, a);
}

// PD above 16 users, 17 to 32 vectors: a wave for each 16 while the chip has a
// SIMD for both, which then take as long as one (MRC, split BF16, 24 vectors,
// one wave / two, us: 512 subcarriers of B = 1024, U = 32: 59 / 54; 100 of B =
// 4096: 212 / 185; 600 of B = 1024, U = 24: 59 / 77).
static bool split_tiles(int W) { return W <= 512; }

template <int NT, int PREC>
static hipError_t launch_lmmse(const FwdArgs &a, bool fd, hipStream_t s) {
  if (!fd) {
    FwdArgs b = a;
    b.spw = pd_share(a.W, sym_pd_per<NT>());
    const dim3 grid((a.W + b.spw - 1) / b.spw, (a.nsym + 15) / 16);
    if (NT == 2 && a.nsym > 16 && !split_tiles(a.W))
      hipLaunchKernelGGL((eq_symbols_pd_kernel<NT, NT, PREC>), dim3(grid.x), dim3(64), 0, s, b);
    else
      hipLaunchKernelGGL((eq_symbols_pd_kernel<NT, 1, PREC>), grid, dim3(64), 0, s, b);
    return hipGetLastError();
  }
  // waves per subcarrier: its rounds of clusters, at most 2 (16 users) or 4.
  // 14 vectors of 1,200 subcarriers of B = 1024, C = 16, U = 32 take 282 us
  // with one wave each, 230 with two, 191 with four (4,800 of them 716, 709,
  // 684); of 9,600 of B = 256, C = 8, U = 16, 196, 182 and 182
  const int rounds = (a.C * NT + 3) / 4;
  const int nw = waves_in_launch(a.W, rounds == 1 ? 1 : NT == 1 || rounds <= 3 ? 2 : 4);
  if (nw == 1)
    launch_fd<NT, PREC, 1>(a, s);
  else if (nw == 2)
    launch_fd<NT, PREC, 2>(a, s);
  else
    launch_fd<NT, PREC, NT == 1 ? 2 : 4>(a, s);
  return hipGetLastError();
}

template <int NT, int PREC, int M>
static hipError_t launch_direct(const FwdArgs &a, bool fd, hipStream_t s) {
  if (!fd) {
    // the systems of an item share nothing but the start of a stream, which
    // short ones notice (32,768 of B = 64: 100 us with four each, 105 with
    // one; 16,384 of B = 256: 220 and 197)
    FwdArgs b = a;
    b.spw = a.B >= 256 && a.W < (1 << 26) ? 1 : pd_share(a.W, sym_pd_per<NT>());
    const dim3 grid((a.W + b.spw - 1) / b.spw, (a.nsym + 15) / 16);
    if (NT == 2 && a.nsym > 16 && !split_tiles(a.W))
      hipLaunchKernelGGL((eq_direct_pd_kernel<NT, NT, PREC, M>), dim3(grid.x), dim3(64), 0, s, b);
    else
      hipLaunchKernelGGL((eq_direct_pd_kernel<NT, 1, PREC, M>), grid, dim3(64), 0, s, b);
  } else if (a.C > 1 && waves_in_launch(a.W, 2) == 2) {
    hipLaunchKernelGGL((eq_direct_fd_kernel<NT, PREC, M, 2>), dim3(a.W), dim3(128), 0, s, a);
  } else {
    hipLaunchKernelGGL((eq_direct_fd_kernel<NT, PREC, M, 1>), dim3(a.W), dim3(64), 0, s, a);
  }
  return hipGetLastError();
}

template <int NT, int PREC>
static hipError_t launch_tile(const FwdArgs &a, bool fd, bool lama, hipStream_t s) {
  if (!lama) return a.eqz == EQZ_MRC ? launch_direct<NT, PREC, 0>(a, fd, s) : launch_lmmse<NT, PREC>(a, fd, s);
  switch (a.lama_m) {
    case 2: return launch_direct<NT, PREC, 2>(a, fd, s);
    case 4: return launch_direct<NT, PREC, 4>(a, fd, s);
    case 8: return launch_direct<NT, PREC, 8>(a, fd, s);
    default: return hipErrorInvalidValue;
  }
}

int symbol_tile(int U, bool fd) { return 16 * sym_tiles(ut_for(U), fd); }

static hipError_t launch_any(const FwdArgs &a, bool fd, int prec, bool lama, hipStream_t s) {
  if (prec != PREC_FP32 && prec != PREC_BF16X3_NR) return hipErrorInvalidValue;
  if (a.nsym < 1 || a.nsym > symbol_tile(a.U, fd)) return hipErrorInvalidValue;
  if (ut_for(a.U) == 16)
    return prec == PREC_FP32 ? launch_tile<1, PREC_FP32>(a, fd, lama, s) : launch_tile<1, PREC_BF16X3_NR>(a, fd, lama, s);
  return prec == PREC_FP32 ? launch_tile<2, PREC_FP32>(a, fd, lama, s) : launch_tile<2, PREC_BF16X3_NR>(a, fd, lama, s);
}

hipError_t launch_symbols_lama(const FwdArgs &a, bool fd, int prec, hipStream_t s) { return launch_any(a, fd, prec, true, s); }

hipError_t launch_symbols(const FwdArgs &a, bool fd, int prec, hipStream_t s) { return launch_any(a, fd, prec, false, s); }

}  // namespace dbpeq
