// Gram and matched filters of up to 16 (32) receive vectors per channel matrix
// in 16 x 16 tiles, in one pass over H: the stream of the several-vector
// kernels (eq_symbols.hip) and of LAMA vector by vector (eq_lama.hip).
//
// Tile layout.  Everything runs in 16 x 16 tiles: NT = 1 or 2 tiles of users
// (U <= 16, U <= 32) and NC = 1 or 2 of symbols.  Lane (g, c) = (lane / 16, lane % 16)
// loads rows of its group for user c (and 16 + c) of H and symbol c (and 16 + c): the
// A and B operands of the products over rows.  Of the Gram matrix only the
// blocks (0, 0), (1, 0) and (1, 1) are formed (seven real FP32 products at 32
// users where full 32 x 32 tiles take eight, and twice the symbols).  Results
// come in MFMA accumulator layout, lane (kk, c) holding rows 4 kk + r of
// column c.
#pragma once
#include "eq_round.h"

namespace dbpeq {

// ---------------------------------------------------------------- streaming
// Rows per lane group and row block.  At 16 users two blocks of eight rows
// take 64 registers, of four 32: FD, whose solves bound it, runs a wave more
// per SIMD with four (14 vectors, 9,600 subcarriers of B = 256, U = 16, C = 8:
// 166 -> 159 us; C = 16: 311 -> 235).  PD streams, and wants the bytes in
// flight (300 subcarriers: 54 us with eight rows, 58 with four).
constexpr int sym_rows(int NT, bool fd) { return NT == 1 && !fd ? 8 : 4; }
// Row e of lane group g within the block (the products sum over rows: any
// order will do that H and Y share).  At 16 users the rows go to the groups in
// pairs: a 16-byte load of Y then covers two rows, and the four groups 64
// consecutive bytes of a vector (14 vectors, PD 38,400 / 4 subcarriers of B =
// 256, U = 16: 113 against 121 us with eight rows per group; at 32 users, with
// half the rows, it was 5% slower).
template <int NT>
__device__ __forceinline__ constexpr int tile_row(int e, int g) {
  return NT == 1 ? 8 * (e / 2) + 2 * g + e % 2 : 4 * g + e;
}

struct TileSlot {
  float2 h[8];  // row e of the group: h[e], or h[2 e] and h[2 e + 1] (users c, 16 + c)
  float2 y[8];  // row e: y[NC e + n] (symbol 16 n + c)
  int s;
  int nv;     // rows from the group's first to the end of the system
  bool full;  // the whole block is inside the system
  bool last;
};

template <int NT>
struct TileOff {
  unsigned h, h1;  // users c and 16 + c of the group's first row, or out of range
  unsigned y, y1;  // the same row of symbols c and 16 + c < nsym, else out of range
  int row;         // the group's first row within a block
};

template <int NT>
__device__ __forceinline__ TileOff<NT> tile_offsets(int U, int B, int nsym) {
  const int lane = lane_id();
  const int c = lane % 16, row = tile_row<NT>(0, lane / 16);
  TileOff<NT> o;
  o.h = c < U ? (unsigned)((row * U + c) * 8) : kOutOfRange;
  o.h1 = 16 + c < U ? (unsigned)((row * U + 16 + c) * 8) : kOutOfRange;
  o.y = c < nsym ? (unsigned)(((unsigned)c * (unsigned)B + (unsigned)row) * 8u) : kOutOfRange;
  o.y1 = 16 + c < nsym ? (unsigned)((16u + (unsigned)c) * (unsigned)B + (unsigned)row) * 8u : kOutOfRange;
  o.row = row;
  return o;
}

// Loads the row block at rb of rows [r0, r1) of H (row stride U) and of the
// tile's receive vectors (vector stride B, Yw = vector 0 of the tile).  The Y
// descriptor spans from row r0 of the first vector to row r1 of the last one:
// rows past r1 of the other vectors are in range and are masked by nv when
// the block is consumed.  Each load is wholly inside or wholly outside its
// descriptor (the 16-byte loads are those of full blocks).  The loads of Y
// use the default policy: they share cache lines (with the nontemporal one
// the lines were fetched again, 22-28% more bytes than the algorithm reads).
template <int NT, int NC, int E>
__device__ __forceinline__ void load_tile_slot(TileSlot &b, const TileOff<NT> &lo, const float2 *__restrict__ Hw,
                                               const float2 *__restrict__ Yw, int U, int B, int nsym, int rb,
                                               int r0, int r1, bool live) {
  const int nrow = live ? r1 - r0 : 0;
  const int ylen = live ? ((nsym - 1) * B + (r1 - r0)) * 8 : 0;
  const __amdgpu_buffer_rsrc_t rh =
      __builtin_amdgcn_make_buffer_rsrc((void *)(Hw + (size_t)r0 * U), (short)0, nrow * U * 8, kBufFlags);
  const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void *)(Yw + r0), (short)0, ylen, kBufFlags);
  const unsigned rowb = (unsigned)((rb - r0) * U * 8);
  const unsigned step = (unsigned)(U * 8);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if constexpr (NT == 1) {
      b.h[e] = buf_ld2<kLoadLast>(rh, lo.h + rowb + tile_row<NT>(e, 0) * step);
    } else {
      b.h[2 * e] = buf_ld2<kLoadLast>(rh, lo.h + rowb + tile_row<NT>(e, 0) * step);
      b.h[2 * e + 1] = buf_ld2<kLoadLast>(rh, lo.h1 + rowb + tile_row<NT>(e, 0) * step);
    }
  }
  const unsigned yb = (unsigned)((rb - r0) * 8);
  b.full = live && rb + 4 * E <= r1;
  if (NT == 1 && b.full) {
#pragma unroll
    for (int e = 0; e < E; e += 2) {
      const f4 v = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(ry, lo.y + yb + 8u * tile_row<NT>(e, 0), 0, kLoadKeep));
      b.y[e] = make_float2(v.x, v.y);
      b.y[e + 1] = make_float2(v.z, v.w);
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      b.y[NC * e] = buf_ld2<kLoadKeep>(ry, lo.y + yb + 8u * tile_row<NT>(e, 0));
      if constexpr (NC == 2) b.y[2 * e + 1] = buf_ld2<kLoadKeep>(ry, lo.y1 + yb + 8u * tile_row<NT>(e, 0));
    }
  }
  b.nv = r1 - (rb + lo.row);
}

// ---------------------------------------------------------------- Gram and matched filters
// Accumulators of the Gram blocks 0 = (0, 0), 1 = (1, 0), 2 = (1, 1).  FP32:
// rr = P = (Hr + Hi)^T (Hr + Hi) and ri = Hr^T Hi; block 1 also ir = Hi^T Hr
// (the diagonal blocks take it from the transpose of ri).  Split BF16: rr, ii
// and ri, block 1 also ir.
template <int NT>
struct TileAcc {
  f4 rr[2 * NT - 1], ri[2 * NT - 1], ii[2 * NT - 1], ir;
};
// Matched filters.  FP32 forms H^H Y with three real products (Gauss):
//   k1 = (Hr - Hi)^T Yr,  k2 = Hr^T (Yi - Yr),  k3 = Hi^T (Yr + Yi),
//   Re M = k1 + k3,   Im M = k1 + k2;
// the split-BF16 form accumulates Re M in k1 and Im M in k2 directly.
template <int NT, int NC>
struct TileMf {
  f4 k1[NT][NC], k2[NT][NC], k3[NT][NC];
};

template <int NT, int NC>
__device__ __forceinline__ void tile_zero(TileAcc<NT> &a, TileMf<NT, NC> &m) {
  const f4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int b = 0; b < 2 * NT - 1; ++b) a.rr[b] = a.ri[b] = a.ii[b] = z;
  a.ir = z;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int n = 0; n < NC; ++n) m.k1[t][n] = m.k2[t][n] = m.k3[t][n] = z;
}

// BF16 operands of one row block of E rows per lane: 8 (K = 32) or 4 (K = 16).
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
template <int E>
using BfVec = std::conditional_t<E == 8, bf8, bf4>;
__device__ __forceinline__ f4 mma16(bf4 a, bf4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4, a), __builtin_bit_cast(s4, b), c, 0, 0, 0);
}

template <int E>
struct Split {
  BfVec<E> h, l;
};
// acc += a b with both operands split: hi lo + lo hi + hi hi
template <int E>
__device__ __forceinline__ f4 mma_split(const Split<E> &a, const Split<E> &b, f4 c) {
  c = mma16(a.h, b.l, c);
  c = mma16(a.l, b.h, c);
  return mma16(a.h, b.h, c);
}

template <int NT, int NC, int PREC, int E>
__device__ __forceinline__ void gram_mf_tile(TileSlot &sl, TileAcc<NT> &acc, TileMf<NT, NC> &m) {
  if (!sl.full) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (tile_row<NT>(e, 0) >= sl.nv)
#pragma unroll
        for (int n = 0; n < NC; ++n) sl.y[NC * e + n] = make_float2(0.f, 0.f);
  }
  if constexpr (PREC == PREC_FP32) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float yre[NC], ydif[NC], ysum[NC];
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        const float2 y = sl.y[NC * e + n];
        yre[n] = y.x;
        ydif[n] = y.y - y.x;
        ysum[n] = y.x + y.y;
      }
      float sum[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float2 h = sl.h[NT * e + t];
        sum[t] = h.x + h.y;
        acc.rr[2 * t] = mma32(sum[t], sum[t], acc.rr[2 * t]);
        m.k1[t][0] = mma32(h.x - h.y, yre[0], m.k1[t][0]);
        acc.ri[2 * t] = mma32(h.x, h.y, acc.ri[2 * t]);
        m.k2[t][0] = mma32(h.x, ydif[0], m.k2[t][0]);
        m.k3[t][0] = mma32(h.y, ysum[0], m.k3[t][0]);
        if constexpr (NC == 2) {
          m.k1[t][1] = mma32(h.x - h.y, yre[1], m.k1[t][1]);
          m.k2[t][1] = mma32(h.x, ydif[1], m.k2[t][1]);
          m.k3[t][1] = mma32(h.y, ysum[1], m.k3[t][1]);
        }
      }
      if constexpr (NT == 2) {
        const float2 h0 = sl.h[2 * e], h1 = sl.h[2 * e + 1];
        acc.rr[1] = mma32(sum[1], sum[0], acc.rr[1]);
        acc.ri[1] = mma32(h1.x, h0.y, acc.ri[1]);
        acc.ir = mma32(h1.y, h0.x, acc.ir);
      }
    }
  } else if constexpr (NC == 2) {
    static_assert(PREC == PREC_BF16X3_NR && E == 4, "one-pass forms only");
    // Four rows are half of the k = 32 of a product, and k = 16 ones run at half
    // the rate, which bounds this form.  Real and imaginary part side by side
    // fill it where their products are summed: Re G, Re M = [Hr Hi]^T [Yr; Yi],
    // Im M = [Hr Hi]^T [Yi; -Yr].  The squares on the diagonal of G add up, and
    // so does the rounding of their sum: rr and ii keep sums of half as many
    // (one sum of all: 0.7% more error in the MRC estimates of B = 1024).  With
    // one symbol tile FD lost a wave per SIMD to the registers that this takes.
    // MRC of 24 vectors, PD, 600 subcarriers of B = 1024, U = 24: 67 and 59 us.
    Split<8> h[NT], y[NC], w[NC];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float2 v = sl.h[NT * e + t];
        h[t].h[e] = (__bf16)v.x;
        h[t].l[e] = (__bf16)(v.x - (float)h[t].h[e]);
        h[t].h[4 + e] = (__bf16)v.y;
        h[t].l[4 + e] = (__bf16)(v.y - (float)h[t].h[4 + e]);
      }
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        const float2 v = sl.y[NC * e + n];
        y[n].h[e] = w[n].h[4 + e] = (__bf16)v.x;
        y[n].l[e] = w[n].l[4 + e] = (__bf16)(v.x - (float)y[n].h[e]);
        y[n].h[4 + e] = w[n].h[e] = (__bf16)v.y;
        y[n].l[4 + e] = w[n].l[e] = (__bf16)(v.y - (float)y[n].h[4 + e]);
        // round-to-nearest-even is symmetric: the split of -yr is the negated split
        w[n].h[4 + e] = -w[n].h[4 + e];
        w[n].l[4 + e] = -w[n].l[4 + e];
      }
    }
    auto part = [](const Split<8> &v, auto Im) {
      constexpr int k = 4 * decltype(Im)::value;
      return Split<4>{__builtin_shufflevector(v.h, v.h, k, k + 1, k + 2, k + 3),
                      __builtin_shufflevector(v.l, v.l, k, k + 1, k + 2, k + 3)};
    };
    constexpr std::integral_constant<int, 0> Re{};
    constexpr std::integral_constant<int, 1> Im{};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const Split<4> re = part(h[t], Re), im = part(h[t], Im);
      acc.rr[2 * t] = mma16(h[t].h, h[t].l, acc.rr[2 * t]);
      acc.ii[2 * t] = mma16(h[t].l, h[t].h, acc.ii[2 * t]);
      acc.rr[2 * t] = mma16(re.h, re.h, acc.rr[2 * t]);
      acc.ii[2 * t] = mma16(im.h, im.h, acc.ii[2 * t]);
      acc.ri[2 * t] = mma_split<4>(re, im, acc.ri[2 * t]);
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        m.k1[t][n] = mma_split<8>(h[t], y[n], m.k1[t][n]);
        m.k2[t][n] = mma_split<8>(h[t], w[n], m.k2[t][n]);
      }
    }
    if constexpr (NT == 2) {
      acc.rr[1] = mma_split<8>(h[1], h[0], acc.rr[1]);
      acc.ri[1] = mma_split<4>(part(h[1], Re), part(h[0], Im), acc.ri[1]);
      acc.ir = mma_split<4>(part(h[1], Im), part(h[0], Re), acc.ir);
    }
  } else {
    static_assert(PREC == PREC_BF16X3_NR, "one-pass forms only");
    Split<E> hr[NT], hi[NT], yr[NC], yi[NC], ny[NC];
#pragma unroll
    for (int e = 0; e < E; ++e) {
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        const float2 y = sl.y[NC * e + n];
        yr[n].h[e] = (__bf16)y.x;
        yr[n].l[e] = (__bf16)(y.x - (float)yr[n].h[e]);
        yi[n].h[e] = (__bf16)y.y;
        yi[n].l[e] = (__bf16)(y.y - (float)yi[n].h[e]);
        // round-to-nearest-even is symmetric: the split of -yr is the negated split
        ny[n].h[e] = -yr[n].h[e];
        ny[n].l[e] = -yr[n].l[e];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float2 h = sl.h[NT * e + t];
        hr[t].h[e] = (__bf16)h.x;
        hr[t].l[e] = (__bf16)(h.x - (float)hr[t].h[e]);
        hi[t].h[e] = (__bf16)h.y;
        hi[t].l[e] = (__bf16)(h.y - (float)hi[t].h[e]);
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc.rr[2 * t] = mma_split<E>(hr[t], hr[t], acc.rr[2 * t]);
      acc.ri[2 * t] = mma_split<E>(hr[t], hi[t], acc.ri[2 * t]);
      acc.ii[2 * t] = mma_split<E>(hi[t], hi[t], acc.ii[2 * t]);
#pragma unroll
      for (int n = 0; n < NC; ++n) {
        m.k1[t][n] = mma_split<E>(hr[t], yr[n], m.k1[t][n]);
        m.k2[t][n] = mma_split<E>(hr[t], yi[n], m.k2[t][n]);
        m.k1[t][n] = mma_split<E>(hi[t], yi[n], m.k1[t][n]);
        m.k2[t][n] = mma_split<E>(hi[t], ny[n], m.k2[t][n]);
      }
    }
    if constexpr (NT == 2) {
      acc.rr[1] = mma_split<E>(hr[1], hr[0], acc.rr[1]);
      acc.ri[1] = mma_split<E>(hr[1], hi[0], acc.ri[1]);
      acc.ii[1] = mma_split<E>(hi[1], hi[0], acc.ii[1]);
      acc.ir = mma_split<E>(hi[1], hr[0], acc.ir);
    }
  }
}

// Complex tiles in accumulator layout (register r of lane (kk, c): row
// 4 kk + r, column c).
template <int N>
struct Tiles {
  f4 re[N], im[N];
};

// Byte offsets of the accumulator positions in 16 x 16 tiles of LDS, the row 4
// kk + r of register r swizzled and added as in GramAddr: [4 kk][c] and its
// transpose of floats, element (4 kk, c) of a packed block.
struct TileAddr {
  uint32_t w, t, p;
};
__device__ __forceinline__ TileAddr tile_addr() {
  const int lane = lane_id();
  const uint32_t i0 = 4 * (lane / 16), c = lane % 16;
  return {4 * (16 * i0 + (c ^ i0)), 4 * (16 * c + (c ^ i0)), 8 * (16 * i0 + (c ^ i0))};
}

// The Gram blocks; the transposes of the diagonal ones go through 256 floats
// of LDS at byte address `scratch`.
template <int NT, int PREC>
__device__ __forceinline__ void tile_gram(const TileAddr &ta, uint32_t scratch, const TileAcc<NT> &a, Tiles<2 * NT - 1> &G) {
  const uint32_t w = scratch + ta.w, tr = scratch + ta.t;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int b = 2 * t;
    wave_sync();
    sfor<4>([&](auto R) {
      constexpr int r = R;
      lds_f((w ^ (4 * r)) + 64 * r) = a.ri[b][r];
    });
    wave_sync();
    sfor<4>([&](auto R) {
      constexpr int r = R;
      const float rij = lds_f(tr ^ (4 * r));
      G.im[b][r] = a.ri[b][r] - rij;
      G.re[b][r] = PREC == PREC_FP32 ? a.rr[b][r] - a.ri[b][r] - rij : a.rr[b][r] + a.ii[b][r];
    });
  }
  if constexpr (NT == 2) {
    G.im[1] = a.ri[1] - a.ir;
    G.re[1] = PREC == PREC_FP32 ? a.rr[1] - a.ri[1] - a.ir : a.rr[1] + a.ii[1];
  }
}

// Matched filters of symbol tile n.
template <int NT, int PREC, int NC>
__device__ __forceinline__ void tile_mf(const TileMf<NT, NC> &m, int n, Tiles<NT> &M) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    M.re[t] = PREC == PREC_FP32 ? m.k1[t][n] + m.k3[t][n] : m.k1[t][n];
    M.im[t] = PREC == PREC_FP32 ? m.k1[t][n] + m.k2[t][n] : m.k2[t][n];
  }
}

// Gram + matched filters of systems 0..ns-1 (seg(s, Hw, Yw, r0, r1), Yw =
// vector 0 of the tile); done(s, acc, m) follows the last block of system s
// while the next block's loads are in flight.  Two slots (a block is 4 to
// 7.5 KB): with four nothing was faster and LAMA lost a wave (104 against
// 98 us), and one stream over all rounds of an FD wave, which loads the next
// round's first rows during a solve, was 2-8% slower.
template <int NT, int NC, int PREC, int E, class Seg, class Done>
__device__ __forceinline__ void gram_mf_stream(int ns, int U, int B, int nsym, Seg seg, Done done) {
  constexpr int RPB = 4 * E;
  TileAcc<NT> acc;
  TileMf<NT, NC> m;
  tile_zero(acc, m);
  const TileOff<NT> lo = tile_offsets<NT>(U, B, nsym);
  SysRef cur;
  seg(0, cur.Hw, cur.yw, cur.r0, cur.r1);
  cur.s = 0;
  int next = 1;
  int crb = cur.r0;
  bool more = true;
  auto issue = [&](TileSlot &sl) -> bool {
    const bool valid = more;
    load_tile_slot<NT, NC, E>(sl, lo, cur.Hw, cur.yw, U, B, nsym, crb, cur.r0, cur.r1, valid);
    sl.s = cur.s;
    sl.last = crb + RPB >= cur.r1;
    if (valid) {
      if (crb + RPB < cur.r1) {
        crb += RPB;
      } else if (next < ns) {
        seg(next, cur.Hw, cur.yw, cur.r0, cur.r1);
        cur.s = next++;
        crb = cur.r0;
      } else {
        more = false;
      }
    }
    return valid;
  };
  auto consume = [&](TileSlot &b) {
    gram_mf_tile<NT, NC, PREC, E>(b, acc, m);
    if (b.last) {
      done(b.s, acc, m);
      tile_zero(acc, m);
    }
  };
  TileSlot sa, sb;
  issue(sa);
  while (true) {
    const bool vb = issue(sb);
    __builtin_amdgcn_sched_barrier(0);
    consume(sa);
    if (!vb) break;
    const bool va = issue(sa);
    __builtin_amdgcn_sched_barrier(0);
    consume(sb);
    if (!va) break;
  }
}

// Rows of system s of a list: whole subcarriers from w0 (PD), or clusters
// from c0 of subcarrier w0 (FD).
__device__ __forceinline__ auto pd_seg(const FwdArgs &a, int w0) {
  return [&a, w0](int s, const float2 *&Hw, const float2 *&Yw, int &r0, int &r1) {
    const size_t w = (size_t)w0 + s;
    Hw = a.H + w * ((size_t)a.B * a.U);
    Yw = a.y + w * (size_t)a.ysw;
    r0 = 0;
    r1 = a.B;
  };
}
// cluster(s): the s-th of them
template <class Cluster>
__device__ __forceinline__ auto fd_seg(const FwdArgs &a, int w, Cluster cluster) {
  return [&a, w, cluster](int s, const float2 *&Hw, const float2 *&Yw, int &r0, int &r1) {
    Hw = a.H + (size_t)w * ((size_t)a.B * a.U);
    Yw = a.y + (size_t)w * (size_t)a.ysw;
    cluster_rows<FwdArgs>(cluster(s), r0, r1);
  };
}

}  // namespace dbpeq
