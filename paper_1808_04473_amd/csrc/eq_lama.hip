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
// row of G, and iterate one after the other, or take a wave each.
// eq_symbols.hip iterates on all vectors of a system at once, on MFMA: better
// where they are many (lama_per).
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
// Waves per FD workgroup, at most.
constexpr int kLamaWaves = 4;

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
  // 0 times the entries: NaN if one of them is not finite
  float qx = 0.f, qy = 0.f;
#pragma unroll
  for (int k = 0; k < UT; ++k) {
    const float2 g = lds_el<UT>(sm.A[slot], i, k);
    qx = fmaf(g.x, 0.f, qx);
    qy = fmaf(g.y, 0.f, qy);
    f.x[k] = make_float2(g.x * scale, -g.y * scale);
  }
  const float2 m = sm.M[0][slot][i];
  return gany<UT>(!(qx == 0.f && qy == 0.f) || (one && !finite2(m)));
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

// Vectors v0 .. v0+nv-1 of subcarriers w0 .. w0+nvalid-1.
template <int UT, int PREC, int M, int NV>
__device__ __forceinline__ void lama_pd_task(const FwdArgs &a, int w0, int nvalid, int v0, int nv, const LamaLds<UT> &sm) {
  const int lane = lane_id();
  const int g = lane / UT, i = lane % UT;
  const size_t HB = (size_t)a.B * a.U;
  auto seg = [&](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
    const size_t w = (size_t)w0 + s;
    Hw = a.H + w * HB;
    yw = a.y + w * (size_t)a.ysw + (size_t)v0 * a.B;
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
      const size_t at = (size_t)w * a.zsw + (size_t)(v0 + n) * a.U + i;
      a.z[at] = bad ? make_float2(nanv, nanv) : o.z;
      if (a.s2) a.s2[at] = bad ? nanv : o.s2;
    }
  }
  if (live && i == 0 && v0 == 0 && a.info) a.info[w] = bad ? -1 : 0;
}

// Vectors v0 .. v0+nv-1 of subcarrier w, all its clusters: the nw waves of the
// workgroup take the rounds in turn.
template <int UT, int PREC, int M, int NV>
__device__ __forceinline__ void lama_fd_task(const FwdArgs &a, int w, int v0, int nv, const LamaLds<UT> &sm, int wv, int nw, int ldsv) {
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
  for (int base = wv * NSYS; base < C; base += nw * NSYS) {
    const int nvalid = min(NSYS, C - base);
    auto seg = [&](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
      Hw = a.H + (size_t)w * HB;
      yw = a.y + (size_t)w * a.ysw + (size_t)v0 * a.B;
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
    if (live && i == 0 && v0 == 0 && a.info) a.info[(size_t)w * C + c] = bad ? -1 : 0;
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
  if (nw > 1) {
    // the waves' sums meet in wave order
    float *part = &sm.A[0][0][0].x;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      part[(3 * k) * 64 + lane] = tk[k];
      part[(3 * k + 1) * 64 + lane] = zx[k];
      part[(3 * k + 2) * 64 + lane] = zy[k];
    }
    __syncthreads();
    if (wv != 0) return;
    for (int q = 1; q < nw; ++q) {
      const float *o = part + q * (lama_lds_bytes<UT>(ldsv) / sizeof(float));
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        tk[k] += o[(3 * k) * 64 + lane];
        zx[k] += o[(3 * k + 1) * 64 + lane];
        zy[k] += o[(3 * k + 2) * 64 + lane];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int n = g + NSYS * k;
    if (n >= nv || i >= a.U) continue;
    const float inv = 1.0f / tk[k];
    const size_t at = (size_t)w * a.zsw + (size_t)(v0 + n) * a.U + i;
    a.z[at] = user_nu ? make_float2(zx[k], zy[k]) : make_float2(zx[k] * inv, zy[k] * inv);
    if (a.s2) a.s2[at] = user_nu ? tk[k] : inv;
  }
}

// PD: one wave per workgroup, `spw` subcarriers.  FD: blockDim / 64 waves, one
// subcarrier.  Block row y takes lama_per receive vectors, at most NV.
// Occupancy, waves per SIMD.  UT = 16: 3 (the row of G, the iterates and the
// denoiser's level terms spill at 4), UT = 32: 2.  And no more than 4 and 2 even
// where registers and LDS would hold a few more waves on a CU: those spread
// unevenly over the SIMDs (FD, 2,500 subcarriers of B = 512, U = 20, C = 8: 122 us
// against 103; PD, 20,000 of B = 64, U = 8: 32 against 28).
template <int UT, int PREC, bool FD, int M, int NV>
__global__ __launch_bounds__(64 * (FD ? kLamaWaves : 1)) __attribute__((amdgpu_waves_per_eu(UT == 16 ? 3 : 2, UT == 16 ? 4 : 2))) void eq_lama_kernel(const FwdArgs a) {
  extern __shared__ __align__(128) float2 lama_lds[];
  const int ldsv = NV < kLamaTile ? NV : a.lama_per;
  const int wv = FD ? __builtin_amdgcn_readfirstlane(threadIdx.x / 64) : 0, nw = FD ? blockDim.x / 64 : 1;
  float2 *base = lama_lds + wv * (lama_lds_bytes<UT>(ldsv) / sizeof(float2));
  const LamaLds<UT> sm = {reinterpret_cast<float2 (*)[UT][UT]>(base),
                          reinterpret_cast<float2 (*)[64 / UT][UT]>(base + (64 / UT) * UT * UT)};
  const int per = NV == 1 ? 1 : a.lama_per;
  const int v0 = per * blockIdx.y, nv = NV == 1 ? 1 : min(per, a.nsym - v0);
  if constexpr (FD) {
    lama_fd_task<UT, PREC, M, NV>(a, blockIdx.x, v0, nv, sm, wv, nw, ldsv);
  } else {
    const int w0 = blockIdx.x * a.spw;
    lama_pd_task<UT, PREC, M, NV>(a, w0, min(a.spw, a.W - w0), v0, nv, sm);
  }
}

// PD systems per wave.  Where one each would be a wave or two per SIMD, many
// iterations want one wave with more of its lane groups at work: 1,200
// subcarriers of B = 256, U = 16, 3 vectors of 64-QAM, 40 iterations took 137 us
// with one system each, 88 with two.
static int lama_pd_share(const FwdArgs &a) {
  const bool few = a.W <= kPdItems && a.W > kPdItems / 2 && a.nsym * a.lama_t > 40;
  return pd_share(a.W, 64 / ut_for(a.U), few ? kPdItems / 2 : kPdItems);
}

// Waves of an FD subcarrier: one for each of its rounds while the chip has room
// for them (64 subcarriers of B = 256, U = 16, C = 8, 2 vectors of 64-QAM, 10
// iterations: 17.5 us with two, 23.3 with one; 600 of B = 1,024, U = 24, C = 16,
// 4 vectors: 215 with four, 396 with one); the limit is a little over the
// waves that run at once (2,000 of B = 512, U = 20, C = 8, one vector, 1
// iteration: 66 with two, 62 with one).
static int lama_fd_waves(const FwdArgs &a) {
  const int rounds = (a.C * ut_for(a.U) + 63) / 64, most = (a.U > 16 ? 3 : 4) * kPdItems / 2;
  int nw = 1;
  while (nw < kLamaWaves && 2 * nw <= rounds && a.W <= most / (2 * nw)) nw *= 2;
  return nw;
}

// Vectors that a wave takes, sharing its pass over H: all of the call, or one
// (each vector a row of blocks, which pass over H again, from the caches); 0 if
// the tile is faster.  The costs, in iterations of one lane group on one
// vector, of a SIMD: its waves (at least one) times the pass, in proportion to
// the rows of H, and the iterations of all its lane groups, also idle ones; an
// iteration of a tile takes as long as 10 to 14, by the levels of its denoiser,
// for any number of vectors.  A tile's pass, and the lane groups' one of more
// than 4 vectors (2 above 16 users), whose matched filters come from the tiles,
// load less at a time, which a second wave on the SIMD hides.  Above 8 vectors and 16 users LDS holds 7 waves a CU, and
// registers 8.  Fitted to 3,500 calls of 35 sizes, where it picks the fastest
// or one 0.5% slower on average.  Tile / all vectors / one, us, at 64-QAM: PD, 300
// subcarriers of B = 256, U = 16, 4 vectors, 10 iterations 30 / 35 / 21; 8, 4: 19 /
// 35 / 22; 4,800 of them, 8, 4: 64 / 86 / 203; 2, 10: 104 / 55 / 76.  FD, 4,800 of B =
// 256, C = 8, U = 16: 4, 2: 108 / 87 / 139; 10, 10: 581 / 547 / 641; 14, 10: 581 / 876 /
// 896; 300 of them, 8, 10: 128 / 96 / 45.
static int lama_per(const FwdArgs &a, bool fd) {
  const int n = a.nsym;
  if (n == 1) return 1;
  if (n > kLamaTile) return 0;
  const bool u32 = a.U > 16;
  const int groups = 64 / ut_for(a.U), sys = fd ? a.C : lama_pd_share(a);
  const int held = (sys + groups - 1) / groups * groups;  // systems, idle lane groups included
  const int nw = fd ? lama_fd_waves(a) : 1;
  const float waves = fd ? a.W : (a.W + sys - 1) / sys, rows = fd ? a.B : (float)a.B * sys;
  auto load = [](float w) { return w > kPdItems / 2 ? w / (kPdItems / 2) : 1.0f; };
  const bool full = waves > kPdItems, wide_full = waves * nw > kPdItems;
  const float pass = (u32 ? 0.2f : 0.1f) * rows;
  const float tile_pass = (u32 ? (full ? 0.29f : 0.21f) : full ? 0.19f : 0.15f) * rows;
  const float wide_pass = (u32 ? 0.3f : wide_full ? 0.19f : 0.33f) * rows;
  const float tile_it = (u32 ? 8.1f + 0.7f * a.lama_m : 9.6f + 0.31f * a.lama_m) * sys;
  const float its = (float)a.lama_t * held;
  const float tile = load(waves) * (tile_pass + tile_it * (a.lama_t - 1));
  const float one = load(waves * nw * n) * (pass + its) / nw;
  const float all = load(waves * nw) * (u32 && n > 8 ? 1.5f : 1.0f) * ((n > (u32 ? 2 : 4) ? wide_pass : pass) + n * its) / nw;
  if (tile < one && tile < all) return 0;
  return one < all ? 1 : n;
}

bool lama_by_vector(const FwdArgs &a, bool fd) { return lama_per(a, fd) != 0; }

template <int UT, int PREC, bool FD, int M, int NV>
static hipError_t launch_lama_one(const FwdArgs &a, hipStream_t s) {
  FwdArgs b = a;
  b.spw = FD ? 1 : lama_pd_share(a);
  b.lama_per = lama_per(a, FD);
  const int nw = FD ? lama_fd_waves(a) : 1;
  const dim3 grid((a.W + b.spw - 1) / b.spw, (a.nsym + b.lama_per - 1) / b.lama_per);
  hipLaunchKernelGGL((eq_lama_kernel<UT, PREC, FD, M, NV>), grid, dim3(64 * nw),
                     nw * lama_lds_bytes<UT>(NV < kLamaTile ? NV : b.lama_per), s, b);
  return hipGetLastError();
}

template <int UT, int PREC, bool FD, int M>
static hipError_t launch_lama_nv(const FwdArgs &a, hipStream_t s) {
  // the narrowest form that holds the vectors of a wave
  const int per = lama_per(a, FD);
  if (per == 1) return launch_lama_one<UT, PREC, FD, M, 1>(a, s);
  if (per == 2) return launch_lama_one<UT, PREC, FD, M, 2>(a, s);
  if constexpr (UT == 16)
    if (per <= 4) return launch_lama_one<UT, PREC, FD, M, 4>(a, s);
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
  if (a.nsym < 1 || !lama_by_vector(a, fd)) return hipErrorInvalidValue;
  const int UT = ut_for(a.U);
  if (UT == 16) return fd ? launch_lama_prec<16, true>(a, prec, s) : launch_lama_prec<16, false>(a, prec, s);
  return fd ? launch_lama_prec<32, true>(a, prec, s) : launch_lama_prec<32, false>(a, prec, s);
}

}  // namespace dbpeq
