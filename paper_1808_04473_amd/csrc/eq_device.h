// Device building blocks of the equaliser kernels (gfx950, wave64).
//
// Work decomposition.  A wave owns a "round" of NSYS = 64/UT small systems
// (UT = 16 or 32 is the padded user count).  Two layouts are used:
//
//  * streaming layout (Gram + matched filter): lane l covers column
//    col = l % UT of H and row offset g = l / UT.  One load step reads
//    RPS = 64/UT consecutive rows of H (RPS*U*8 contiguous bytes) with one
//    8-byte load per lane.  The loaded value is at the same time the A and B
//    operand of an MFMA whose K index runs over rows, so H_c^H H_c needs no
//    LDS staging: FP32 MFMA consumes one load step per instruction
//    (16x16x4 / 32x32x2), BF16 MFMA eight (16x16x32 / 32x32x16).
//
//  * solve layout: lane l works on system s = l / UT, row / column
//    i = l % UT.  Lane i owns row i of the Cholesky factor L and then, in the
//    same registers, column i of X = L^{-1} (solve_slot), so
//    diag(A^{-1})_u = sum_j |X_ju|^2 and z = X^H (L^{-1} m) need no
//    cross-lane reduction.  Values move between lanes of a group by
//    broadcasting one lane: a DPP row broadcast, after a v_permlane16_swap
//    for 32-lane groups, fused into the FMAC that consumes it.
#pragma once
#include <stddef.h>

#include <utility>

#include "eq_common.h"

namespace dbpeq {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- compile-time loops
template <int... Is, class F>
__device__ __forceinline__ void sfor_impl(std::integer_sequence<int, Is...>, F &&f) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void sfor(F &&f) {
  sfor_impl(std::make_integer_sequence<int, N>{}, f);
}

// Lane index within the wave.  Opaque to the optimiser: otherwise every
// lane-dependent value (masks, offsets, selects) is computed once and kept
// live across the whole kernel, which costs tens of registers; recomputing
// it is one VALU instruction.
__device__ __forceinline__ int lane_id() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

// ---------------------------------------------------------------- cross-lane primitives
// DPP controls (GCN/CDNA data-parallel primitives).
constexpr int DPP_QUAD_XOR1 = 0xB1;      // quad_perm [1,0,3,2]
constexpr int DPP_QUAD_XOR2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int DPP_ROW_MIRROR = 0x140;    // lane i <-> 15 - i inside a row of 16
constexpr int DPP_ROW_HMIRROR = 0x141;   // lane i <-> 7 - i inside half rows
constexpr int DPP_ROW_NEWBCAST = 0x150;  // + k: lane k of each row to the whole row

// Every control used here reads a valid lane, so the bound_ctrl / old value
// never matter; this form lets the compiler fold the DPP into the add (or
// other VOP2 instruction) that consumes it.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Broadcast source of a value v for groups of UT lanes.  A group of 16 lanes
// is one DPP row, so lane K of it is DPP row_newbcast:K of v itself.  A group
// of 32 lanes spans two rows: v_permlane16_swap(v, v) yields `lo`, in which
// the group's first row fills both of its rows, and `hi`, with the second
// row; lane K of the group is then row_newbcast:(K % 16) of lo (K < 16) or
// hi.  One swap serves every K, so a step that broadcasts the same register
// from many lanes pays for it once.
struct BSrc {
  float lo, hi;
};
template <int UT>
__device__ __forceinline__ BSrc bsrc(float v) {
  if constexpr (UT == 16) {
    return {v, v};
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
  }
}
template <int K>
__device__ __forceinline__ float bpick(const BSrc &b) {
  return K < 16 ? b.lo : b.hi;
}

// Value of lane K of this lane's group of UT lanes.
template <int UT, int K>
__device__ __forceinline__ float gbcast(float v) {
  return dpp<DPP_ROW_NEWBCAST + K % 16>(bpick<K>(bsrc<UT>(v)));
}
// acc += (NEG ? -1 : 1) * src[lane K of this lane's DPP row] * b: one VOP2
// FMAC whose src0 comes through a DPP row broadcast (src is a BSrc half, so
// that K = group lane % 16).  Written as inline assembly because the
// compiler folds DPP movs into adds but not into FMACs.  The hardware needs
// two wait states between a VALU write of the DPP source and the read (five
// after a VALU write of EXEC); the compiler does not see the DPP operand of
// inline assembly, so NOP = 4 puts an s_nop 4 at the head of each group of
// these instructions, whose sources are written before the group and not
// inside it.  The build checks the generated assembly for these hazards.
#define EQ_FMAC_ROWBCAST(PRE, NEGS)                                                          \
  asm volatile(PRE "v_fmac_f32_dpp %0, " NEGS "%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" \
               : "+v"(acc)                                                                     \
               : "v"(src), "v"(b), "n"(K))
template <int K, bool NEG, int NOP>
__device__ __forceinline__ void fmac_rowbcast(float &acc, float src, float b) {
  static_assert(NOP == 0 || NOP == 4, "wait states");
  if constexpr (NEG && NOP == 4) EQ_FMAC_ROWBCAST("s_nop 4\n\t", "-");
  else if constexpr (NEG) EQ_FMAC_ROWBCAST("", "-");
  else if constexpr (NOP == 4) EQ_FMAC_ROWBCAST("s_nop 4\n\t", "");
  else EQ_FMAC_ROWBCAST("", "");
}
#undef EQ_FMAC_ROWBCAST

// Sum over the 16 lanes of a DPP row; every lane receives the sum.
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp<DPP_QUAD_XOR1>(v);
  v += dpp<DPP_QUAD_XOR2>(v);
  v += dpp<DPP_ROW_HMIRROR>(v);
  v += dpp<DPP_ROW_MIRROR>(v);
  return v;
}

// Sum of the lane and the one 32 lanes away; both receive it.
__device__ __forceinline__ float xor32_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum / max / any over an aligned group of UT lanes; all lanes get the result.
template <int UT>
__device__ __forceinline__ float gsum(float v) {
  v = row16_sum(v);
  if constexpr (UT == 32) {
    // the two row sums of the 32-lane group, each replicated over the group
    const BSrc r = bsrc<32>(v);
    v = r.lo + r.hi;
  }
  return v;
}
template <int UT>
__device__ __forceinline__ float gmax(float v) {
  v = fmaxf(v, dpp<DPP_QUAD_XOR1>(v));
  v = fmaxf(v, dpp<DPP_QUAD_XOR2>(v));
  v = fmaxf(v, dpp<DPP_ROW_HMIRROR>(v));
  v = fmaxf(v, dpp<DPP_ROW_MIRROR>(v));
  if constexpr (UT == 32) {
    const BSrc r = bsrc<32>(v);
    v = fmaxf(r.lo, r.hi);
  }
  return v;
}
template <int UT>
__device__ __forceinline__ bool gany(bool p) {
  const unsigned long long m = __ballot(p);
  const int s = lane_id() / UT;
  const unsigned long long gm = (UT == 64) ? ~0ull : ((1ull << UT) - 1ull) << (s * UT);
  return (m & gm) != 0ull;
}

// Sum over the four 16-lane groups, lane by lane of a group.
__device__ __forceinline__ float groups_sum(float v) {
  const BSrc r = bsrc<32>(v);
  return xor32_sum(r.lo + r.hi);
}

// Sum over the 64/UT lanes that share a column in the streaming layout.
template <int UT>
__device__ __forceinline__ float colsum(float v) {
  if constexpr (UT == 16) v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}

// ---------------------------------------------------------------- MFMA wrappers
template <int UT> struct Acc;
template <> struct Acc<16> { f4 rr, ri, ii; };
template <> struct Acc<32> { f16v rr, ri, ii; };

__device__ __forceinline__ f4 mma32(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f16v mma32(float a, float b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mma16(bf8 a, bf8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f16v mma16(bf8 a, bf8 b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Position (i, j) of accumulator register r in lane l.
template <int UT>
__device__ __forceinline__ void acc_pos(int l, int r, int &i, int &j) {
  if constexpr (UT == 16) {
    i = 4 * (l >> 4) + r;
    j = l & 15;
  } else {
    i = 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
    j = l & 31;
  }
}

template <int UT>
__device__ __forceinline__ void acc_zero(Acc<UT> &a) {
  constexpr int NR = UT == 16 ? 4 : 16;
#pragma unroll
  for (int r = 0; r < NR; ++r) { a.rr[r] = 0.f; a.ri[r] = 0.f; a.ii[r] = 0.f; }
}

// ---------------------------------------------------------------- wave-uniform tables
// Word p[k] of a table that no kernel writes, for wave-uniform k, as a scalar
// load.  Without the constant address space the compiler reads tables through
// the vector memory path, whose results arrive in order: waiting for one
// entry waits for every load of the stream in flight.
template <class T>
__device__ __forceinline__ T table(const T *p, int k) {
  typedef const T __attribute__((address_space(4))) *cp;
  return ((cp)(uintptr_t)p)[__builtin_amdgcn_readfirstlane(k)];
}

// Rows [r0, r1) of cluster c (wave-uniform) from the 16-bit offsets in the
// launch arguments Args, the kernel's first parameter.  There is no 16-bit
// scalar load, and the address of a by-value argument would put a copy of all
// of them in scratch, so by words of the kernel-argument segment.
template <class Args>
__device__ __forceinline__ void cluster_rows(int c, int &r0, int &r1) {
  typedef const char __attribute__((address_space(4))) *bp;
  typedef const uint32_t __attribute__((address_space(4))) *wp;
  const wp w = (wp)((bp)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(Args, off));
  c = __builtin_amdgcn_readfirstlane(c);
  const uint32_t a = w[c >> 1], b = w[(c + 1) >> 1];
  const bool odd = c & 1;
  r0 = odd ? a >> 16 : a & 0xffffu;
  r1 = odd ? b & 0xffffu : b >> 16;
}

// ---------------------------------------------------------------- row-block streaming
// One block = 8 load steps = 8 * (64/UT) rows of one system, in the
// streaming layout: lane l holds H[rb + e*RPS + g][col] (col = l % UT,
// g = l / UT, e = 0..7).  y is loaded once per row (lane j < RPB holds
// y[rb + j]) and handed to the lanes of a row by a lane shuffle: a per-lane
// copy would cost eight vector-memory instructions for 256 bytes.
struct Blk8 {
  float2 h[8];
};

struct Slot {
  float2 h[8];
  float2 yl;
  const float2 *Hw;
  const float2 *yw;
  int s, rb, r1;  // s: system index within its task
  int tk;         // task the system belongs to
  int g;          // row group of this lane (lane / UT)
  bool last;
};

// One system of a stream: rows [r0, r1) of Hw / yw, identified by (tk, s).
struct SysRef {
  const float2 *Hw;
  const float2 *yw;
  int r0, r1, tk, s;
};

// Loads go through buffer resources that cover exactly the system's rows
// [r0, r1): the hardware returns zero for any offset outside the range, so
// rows past r1 and padded columns (col >= U, given an offset that is always
// out of range) need neither clamping nor masking, and the address of each
// load is one integer add.  No load sits behind a divergent branch, so the
// compiler can wait for one block while the next blocks are in flight.
constexpr int kBufFlags = 0x00020000;  // raw 32-bit buffer, gfx9 format bits
constexpr unsigned kOutOfRange = 0x80000000u;

// Cache policy of a stream's loads: the last read of these bytes uses the
// nontemporal policy (they are not kept in L2 / Infinity Cache); a read that
// a later pass of the same wave repeats uses the default policy.
constexpr int kLoadKeep = 0;
constexpr int kLoadLast = 2;  // NT

template <int AUX>
__device__ __forceinline__ float2 buf_ld2(__amdgpu_buffer_rsrc_t r, unsigned off) {
  typedef float f2v __attribute__((ext_vector_type(2)));
  const f2v v = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX));
  return make_float2(v.x, v.y);
}

// Row of load step e of group g (lane / UT) within a row block: each group
// holds 8 consecutive rows, so that y of those rows sits in the group's own
// DPP row (lanes 0..7 of it) and reaches the other lanes by row broadcast.
__device__ __forceinline__ int slot_row(int e, int g) { return 8 * g + e; }

// Per-lane byte offsets of the streaming layout (constant over a stream).
template <int UT>
struct LaneOff {
  unsigned h;  // (8 g U + col) * 8, or out of range for padded columns
  unsigned y;  // (8 g + c) * 8 for lanes c = lane % 16 < 8, else out of range
  int g;       // row group lane / UT
};

template <int UT>
__device__ __forceinline__ LaneOff<UT> lane_offsets(int U) {
  const int lane = lane_id();
  const int col = lane % UT, g = lane / UT, c = lane % 16;
  LaneOff<UT> o;
  o.h = col < U ? (unsigned)((slot_row(0, g) * U + col) * 8) : kOutOfRange;
  o.y = c < 8 ? (unsigned)(slot_row(c, g) * 8) : kOutOfRange;
  o.g = g;
  return o;
}

// Loads the row block at rb of rows [r0, r1).  live = false gives the
// descriptors zero length: every load is then out of range and returns zero
// without a memory access (the same instructions, no traffic).
template <int UT, int AUX>
__device__ __forceinline__ void load_slot(Slot &b, const LaneOff<UT> &lo, const float2 *__restrict__ Hw,
                                          const float2 *__restrict__ yw, int U, int rb, int r0,
                                          int r1, bool live) {
  const int nrow = live ? r1 - r0 : 0;
  const __amdgpu_buffer_rsrc_t rh =
      __builtin_amdgcn_make_buffer_rsrc((void *)(Hw + (size_t)r0 * U), (short)0, nrow * U * 8, kBufFlags);
  const __amdgpu_buffer_rsrc_t ry =
      __builtin_amdgcn_make_buffer_rsrc((void *)(yw + r0), (short)0, nrow * 8, kBufFlags);
  const unsigned h0 = lo.h + (unsigned)((rb - r0) * U * 8);
  const unsigned step = (unsigned)(U * 8);
#pragma unroll
  for (int e = 0; e < 8; ++e) b.h[e] = buf_ld2<AUX>(rh, h0 + e * step);
  b.yl = buf_ld2<AUX>(ry, lo.y + (unsigned)((rb - r0) * 8));
  b.g = lo.g;
  b.Hw = Hw;
  b.yw = yw;
  b.rb = rb;
  b.r1 = r1;
}

// H[rb + slot_row(e, g)][col] of this lane (zero outside the system).
template <int UT>
__device__ __forceinline__ float2 slot_h(const Slot &b, int e, int) {
  return b.h[e];
}

// y[rb + slot_row(E, g)] of this lane's row in load step E (zero past the
// end): lane E of the DPP row holds it.
template <int UT, int E>
__device__ __forceinline__ float2 slot_y(const Slot &b) {
  return make_float2(dpp<DPP_ROW_NEWBCAST + E>(b.yl.x), dpp<DPP_ROW_NEWBCAST + E>(b.yl.y));
}

// Three-slot ring over row blocks: issue(slot) starts the loads of the next
// block (returning false once the stream is exhausted, after issuing the
// same loads against empty descriptors), body(slot) consumes a block and
// done(slot) follows the last block of each system.  Two blocks are in
// flight while one is consumed (a fourth slot measured no faster at either
// group width, and spills in the refining forms).  sched_barrier keeps each
// block's loads where they are issued: the scheduler must not sink them into
// (or hoist the consumer above) the previous block's arithmetic.
template <class SlotT, class Issue, class Body, class Done>
__device__ __forceinline__ void stream_ring3(Issue &issue, Body &body, Done &done) {
  SlotT sa, sb, sc;
  issue(sa);
  bool vb = issue(sb);
  while (true) {
    const bool vc = issue(sc);
    __builtin_amdgcn_sched_barrier(0);
    body(sa);
    if (sa.last) done(sa);
    if (!vb) break;
    const bool va = issue(sa);
    __builtin_amdgcn_sched_barrier(0);
    body(sb);
    if (sb.last) done(sb);
    if (!vc) break;
    vb = issue(sb);
    __builtin_amdgcn_sched_barrier(0);
    body(sc);
    if (sc.last) done(sc);
    if (!va) break;
  }
}

// Streams the row blocks of a sequence of systems produced by gen (a
// functor bool(SysRef &) returning false at the end of the sequence).
template <int UT, int AUX, class Gen, class Body, class Done>
__device__ __forceinline__ void stream_gen(int U, Gen &gen, Body body, Done done) {
  constexpr int RPB = 8 * (64 / UT);
  SysRef cur;
  if (!gen(cur)) return;
  int crb = cur.r0;
  bool more = true;
  const LaneOff<UT> lo = lane_offsets<UT>(U);
  // Every issue executes the same loads: an exhausted stream issues them
  // against empty descriptors (no memory access) so that the number of loads
  // in flight is the same on every path and the compiler can wait for one
  // block at a time.
  auto issue = [&](Slot &sl) -> bool {
    const bool valid = more;
    load_slot<UT, AUX>(sl, lo, cur.Hw, cur.yw, U, crb, cur.r0, cur.r1, valid);
    sl.s = cur.s;
    sl.tk = cur.tk;
    sl.last = crb + RPB >= cur.r1;
    if (valid) {
      if (crb + RPB < cur.r1) {
        crb += RPB;
      } else {
        SysRef nx;
        if (gen(nx)) {
          cur = nx;
          crb = cur.r0;
        } else {
          more = false;
        }
      }
    }
    return valid;
  };
  stream_ring3<Slot>(issue, body, done);
}

// Fixed list of systems 0..ns-1 described by seg(s, Hw, yw, r0, r1);
// done(s) follows the last block of system s.
template <int UT, int AUX, class Seg, class Body, class Done>
__device__ __forceinline__ void stream_blocks(int ns, int U, Seg seg, Body body, Done done) {
  int next = 0;
  auto gen = [&](SysRef &r) -> bool {
    if (next >= ns) return false;
    seg(next, r.Hw, r.yw, r.r0, r.r1);
    r.tk = 0;
    r.s = next++;
    return true;
  };
  stream_gen<UT, AUX>(U, gen, body, [&](const Slot &sl) { done(sl.s); });
}

// ---------------------------------------------------------------- Gram + matched filter
// acc += real split of the block's H^H H: rr = Hr^T Hr, ri = Hr^T Hi,
// ii = Hi^T Hi in the BF16 forms; in FP32, two products only, rr = P =
// (Hr + Hi)^T (Hr + Hi) = Hr^T Hr + Hi^T Hi + ri + ri^T and ri (Re G needs
// only the sum of the two squares, store_gram takes ri + ri^T back out).
// (mfx, mfy) += partial of sum conj(H[row][col]) y[row].
template <int UT, int PREC>
__device__ __forceinline__ void gram_blk(const Slot &sl, int U, Acc<UT> &acc, float &mfx, float &mfy) {
  Blk8 b;
#pragma unroll
  for (int e = 0; e < 8; ++e) b.h[e] = slot_h<UT>(sl, e, U);
  if constexpr (PREC == PREC_FP32) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float sum = b.h[e].x + b.h[e].y;
      acc.rr = mma32(sum, sum, acc.rr);
      acc.ri = mma32(b.h[e].x, b.h[e].y, acc.ri);
    }
  } else if constexpr (PREC == PREC_BF16) {
    bf8 re, im;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      re[e] = (__bf16)b.h[e].x;
      im[e] = (__bf16)b.h[e].y;
    }
    acc.rr = mma16(re, re, acc.rr);
    acc.ri = mma16(re, im, acc.ri);
    acc.ii = mma16(im, im, acc.ii);
  } else {
    bf8 rh, rl, ih, il;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      rh[e] = (__bf16)b.h[e].x;
      rl[e] = (__bf16)(b.h[e].x - (float)rh[e]);
      ih[e] = (__bf16)b.h[e].y;
      il[e] = (__bf16)(b.h[e].y - (float)ih[e]);
    }
    acc.rr = mma16(rh, rl, acc.rr);
    acc.rr = mma16(rl, rh, acc.rr);
    acc.rr = mma16(rh, rh, acc.rr);
    acc.ri = mma16(rh, il, acc.ri);
    acc.ri = mma16(rl, ih, acc.ri);
    acc.ri = mma16(rh, ih, acc.ri);
    acc.ii = mma16(ih, il, acc.ii);
    acc.ii = mma16(il, ih, acc.ii);
    acc.ii = mma16(ih, ih, acc.ii);
  }
  // conj(h) * y as FMACs whose y operand is the DPP row broadcast of the
  // lane that loaded it
  sfor<8>([&](auto E) {
    constexpr int e = E;
    fmac_rowbcast<e, false, e == 0 ? 4 : 0>(mfx, sl.yl.x, b.h[e].x);
    fmac_rowbcast<e, false, 0>(mfy, sl.yl.y, b.h[e].x);
    fmac_rowbcast<e, false, 0>(mfx, sl.yl.y, b.h[e].y);
    fmac_rowbcast<e, true, 0>(mfy, sl.yl.x, b.h[e].y);
  });
}

// Gram + matched filter of systems 0..ns-1; done(s, acc, mf) receives each
// system's accumulators and this lane's share of its matched filter (the sum
// over the 64/UT lanes of a column, see colsum, is the matched filter).
// AUX is the loads' cache policy (kLoadLast unless a later pass re-reads H).
template <int UT, int PREC, int AUX, class Seg, class Done>
__device__ __forceinline__ void gram_stream(int ns, int U, Seg seg, Done done) {
  Acc<UT> acc;
  acc_zero<UT>(acc);
  float mfx = 0.f, mfy = 0.f;
  stream_blocks<UT, AUX>(
      ns, U, seg, [&](const Slot &b) { gram_blk<UT, PREC>(b, U, acc, mfx, mfy); },
      [&](int s) {
        done(s, acc, make_float2(mfx, mfy));
        acc_zero<UT>(acc);
        mfx = 0.f;
        mfy = 0.f;
      });
}

// Residual pass of the refinement step: for system s (zcf(s) gives z[col]
// of that system) accumulates n = H^H (y - H z) and calls done(s, n) with
// n[col] valid in every lane.
template <int UT, class Seg, class Zc, class Done>
__device__ __forceinline__ void residual_stream(int ns, int U, Seg seg, Zc zcf, Done done) {
  float nx = 0.f, ny = 0.f;
  float2 zc = zcf(0);
  stream_blocks<UT, kLoadLast>(
      ns, U, seg,
      [&](const Slot &b) {
        sfor<8>([&](auto E) {
          constexpr int e = E;
          const float2 h = slot_h<UT>(b, e, U);
          // (H z)_row = sum over the UT lanes of this row of h * z
          const float px = gsum<UT>(h.x * zc.x - h.y * zc.y);
          const float py = gsum<UT>(h.x * zc.y + h.y * zc.x);
          const float2 yv = slot_y<UT, e>(b);
          const float rx = yv.x - px;
          const float ry = yv.y - py;
          nx = fmaf(h.x, rx, nx);
          nx = fmaf(h.y, ry, nx);
          ny = fmaf(h.x, ry, ny);
          ny = fmaf(-h.y, rx, ny);
        });
      },
      [&](int s) {
        done(s, make_float2(colsum<UT>(nx), colsum<UT>(ny)));
        nx = 0.f;
        ny = 0.f;
        if (s + 1 < ns) zc = zcf(s + 1);
      });
}

// Element (i, k) of a UT x UT matrix in LDS.  Rows are not padded: column k
// of row i is stored at k ^ i, so that the lanes of a group that read one
// row, or one column, touch UT different banks.
template <int UT>
__device__ __forceinline__ float2 &lds_el(float2 (*As)[UT], int i, int k) {
  return As[i][k ^ i];
}

// LDS slot of a local solve: the 16 x 16 blocks (0, 0), and for 32 users
// (1, 0) and (1, 1), of the Hermitian matrix, 2 KB each (a third less LDS
// than the full matrix at 32 users: 12 instead of 9 waves per CU).  Swizzled
// like lds_el.
template <int UT>
constexpr int kSlot = UT == 16 ? 256 : 768;
__device__ __forceinline__ float2 &blk_el(float2 *As, int b, int i, int k) {
  return As[256 * b + 16 * i + (k ^ i)];
}

// Orders this wave's LDS accesses before and after the point (they execute
// in order; only the compiler must not move them).  Waves of a workgroup
// that share nothing need no barrier.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// LDS accesses by byte address.
typedef __attribute__((address_space(3))) float lds_f32;
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) f2v lds_f64;
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
__device__ __forceinline__ lds_f32 &lds_f(uint32_t addr) { return *(lds_f32 *)addr; }
__device__ __forceinline__ void lds_put(uint32_t addr, float x, float y) { *(lds_f64 *)addr = f2v{x, y}; }

// Byte offsets, within a packed slot, of the accumulator positions: register
// r holds row i0 + q(r) (i0 from the lane, no bits in common with q) of
// column j, so every swizzled address is one of these with the constant q
// xor-ed into its column bits and added, as an instruction offset, to its row
// bits.  Kept in registers over a stream: formed anew at each system they
// were a tenth of the VALU work of an FD round.
template <int UT>
struct GramAddr {
  uint32_t w, t;  // [i][j] and [j][i] of UT x UT floats
  uint32_t p0;    // element (i, j) of the packed blocks, rows 0..15
  uint32_t p1;    // the same for the rows 16..31 (UT = 32)
  static constexpr int q(int r) { return UT == 16 ? r : 8 * (r >> 2) + (r & 3); }
};
template <int UT>
__device__ __forceinline__ GramAddr<UT> gram_addr() {
  const int lane = lane_id();
  const uint32_t i0 = UT == 16 ? 4 * (lane >> 4) : 4 * (lane >> 5), j = lane % UT;
  GramAddr<UT> o;
  o.w = 4 * (UT * i0 + (j ^ i0));
  o.t = 4 * (UT * j + (j ^ i0));
  o.p0 = 8 * (16 * i0 + ((j & 15) ^ i0));
  o.p1 = o.p0 + 2048 * (1 + (j >> 4));
  return o;
}

// Re G, Im G at the accumulator positions; the transposed ri comes through
// UT x UT floats of LDS at byte address `slot` (aligned to them).
template <int UT, int PREC, int NR>
__device__ __forceinline__ void gram_values(const GramAddr<UT> &ga, uint32_t slot, const Acc<UT> &acc, float (&re)[NR],
                                            float (&im)[NR]) {
  const uint32_t w = slot + ga.w, t = slot + ga.t;
  sfor<NR>([&](auto R) {
    constexpr int r = R, q = GramAddr<UT>::q(r);
    lds_f((w ^ (4 * q)) + 4 * UT * q) = acc.ri[r];
  });
  wave_sync();
  sfor<NR>([&](auto R) {
    constexpr int r = R, q = GramAddr<UT>::q(r);
    const float rij = lds_f(t ^ (4 * q));  // (Hr^T Hi)[j][i]
    im[r] = acc.ri[r] - rij;
    re[r] = PREC == PREC_FP32 ? acc.rr[r] - acc.ri[r] - rij : acc.rr[r] + acc.ii[r];
  });
  wave_sync();
}

// Writes G of one system from the MFMA accumulators into LDS (full Hermitian
// matrix, swizzled rows):
//   Re G = Hr^T Hr + Hi^T Hi,   Im G[i][j] = (Hr^T Hi)[i][j] - (Hr^T Hi)[j][i],
// with Re G = P - ri - ri^T for the two-product FP32 accumulators (see
// gram_blk).  Rows and columns of padded users (i >= U) are zero.
template <int UT, int PREC>
__device__ __forceinline__ void store_gram(float2 (*As)[UT], const Acc<UT> &acc) {
  constexpr int NR = UT == 16 ? 4 : 16;
  const int lane = lane_id();
  float im[NR], re[NR];
  gram_values<UT, PREC>(gram_addr<UT>(), lds_addr(As), acc, re, im);
  sfor<NR>([&](auto R) {
    constexpr int r = R;
    int i, j;
    acc_pos<UT>(lane, r, i, j);
    lds_el<UT>(As, i, j) = make_float2(re[r], im[r]);
  });
}

// The same into the packed slot of the local solves.
template <int UT, int PREC>
__device__ __forceinline__ void store_gram_packed(const GramAddr<UT> &ga, float2 *As, const Acc<UT> &acc) {
  constexpr int NR = UT == 16 ? 4 : 16;
  float im[NR], re[NR];
  const uint32_t slot = lds_addr(As);
  gram_values<UT, PREC>(ga, slot, acc, re, im);
  const uint32_t p0 = slot + ga.p0, p1 = slot + ga.p1;
  const bool low = UT == 16 || lane_id() % 32 < 16;
  sfor<NR>([&](auto R) {
    constexpr int r = R, q = GramAddr<UT>::q(r) & 15;
    if constexpr (UT == 16 || r < 8) {
      // of the rows 0..15 only the block (0, 0) is kept
      if (low) lds_put((p0 ^ (8 * q)) + 128 * q, re[r], im[r]);
    } else {
      lds_put((p1 ^ (8 * q)) + 128 * q, re[r], im[r]);
    }
  });
}

template <int UT>
__device__ __forceinline__ void store_identity(float2 (*As)[UT]) {
  for (int idx = lane_id(); idx < UT * UT; idx += 64) {
    const int i = idx / UT, j = idx % UT;
    lds_el<UT>(As, i, j) = make_float2(i == j ? 1.f : 0.f, 0.f);
  }
}

// ---------------------------------------------------------------- triangular products
// Keeps the scheduler from hoisting the broadcasts of later pivot steps above
// the current one (which would keep hundreds of values live at once).
__device__ __forceinline__ void step_fence() { __builtin_amdgcn_sched_barrier(0); }

// Column i of a UT x UT matrix in lane i.
template <int UT>
struct Columns {
  float2 x[UT];
};

// (X^H t)_u = sum_j conj(X_ju) t_j for lane u; t_j is the DPP row broadcast
// of lane j, fused into the FMACs (t does not change here, so one group).
template <int UT>
__device__ __forceinline__ float2 apply_xh(const Columns<UT> &f, float2 t) {
  const BSrc bx = bsrc<UT>(t.x), by = bsrc<UT>(t.y);
  float r[4] = {0.f, 0.f, 0.f, 0.f};
  sfor<UT>([&](auto J) {
    constexpr int j = J;
    constexpr int p = 2 * (j & 1);
    // the first reader of each source carries the wait states
    fmac_rowbcast<j % 16, false, j == 0 ? 4 : 0>(r[p], bpick<j>(bx), f.x[j].x);
    fmac_rowbcast<j % 16, false, j == 0 ? 4 : 0>(r[p + 1], bpick<j>(by), f.x[j].x);
    fmac_rowbcast<j % 16, false, 0>(r[p], bpick<j>(by), f.x[j].y);
    fmac_rowbcast<j % 16, true, 0>(r[p + 1], bpick<j>(bx), f.x[j].y);
  });
  return make_float2(r[0] + r[2], r[1] + r[3]);
}

__device__ __forceinline__ bool finite2(float2 v) { return isfinite(v.x) && isfinite(v.y); }

// Row sums for the condition estimate and the finiteness test of a system:
// (|Re| + |Im|) of each entry, scaled by 2^-32 so that no row of finite
// entries overflows.  The scaled sum is finite exactly when every entry is,
// and 2^32 times it bounds the row's sum of moduli from above (by at most
// sqrt 2).  Two FMAs per entry, against a square root and two compares.
constexpr float kRowScale = 0x1p-32f;
__device__ __forceinline__ float abs_row_acc(float acc, float2 v) {
  return fmaf(fabsf(v.y), kRowScale, fmaf(fabsf(v.x), kRowScale, acc));
}

// ---------------------------------------------------------------- factor, inverse and solve in one elimination
// Lane i of a group owns row i of A (entries k <= i, zero for k > i) in v[].
// Step J of the right-looking Cholesky A = L L^H subtracts l_iJ conj(l_kJ)
// from a_ik in the lanes i >= k; step J of the inverse X = L^{-1} subtracts
// L_kJ X_Ju from X_ku in the lanes u <= J.  With the columns of X kept
// conjugated both are
//     v[k] -= s conj(l_kJ),   k > J,
// with s = l_iJ in the lanes past J and conj(X_Ju) in the others, and lane J,
// whose row of L is used up after step J, starts column J of X in the
// registers of that row: one set of registers and one pass of FMACs do both.
// The right-hand side rides along: acc_i -= s t_J is the forward
// substitution t = L^{-1} m in the lanes past J and, restarted from zero in
// lane J, -z_u = -sum_J conj(X_Ju) t_J in the others; d_u = sum_J |X_Ju|^2.
//
// Lanes J < i < k take no part in the update of v[k] (lane i must find its
// v[k] zero when its column starts): EXEC leaves them out.  It is set by
// scalar moves inside the assembly block, which do not take vector issue
// slots, and is all ones again at its end.  Callers run in wave-uniform
// control flow with all 64 lanes active.

// Lanes of each UT-lane group with index >= k, over 32 lanes.
template <int UT>
constexpr uint32_t lanes_ge(int k) {
  if (UT == 32) return k >= 32 ? 0u : ~0u << k;
  const uint32_t p = k >= 16 ? 0u : (0xffffu << k) & 0xffffu;
  return p | p << 16;
}
// A lane predicate from its 32-lane pattern (the same in both halves of the
// wave).  The scalar moves are volatile: as plain constants the compiler
// keeps every pattern of the elimination live, and spills them.
__device__ __forceinline__ bool lanes(uint32_t pattern) {
  uint32_t lo, hi;
  asm volatile("s_mov_b32 %0, %2\n\ts_mov_b32 %1, %2" : "=s"(lo), "=s"(hi) : "n"(pattern));
  return __builtin_amdgcn_inverse_ballot_w64((uint64_t)hi << 32 | lo);
}

// v[k] -= s conj(b_k) for N consecutive columns from K0 (b_k: lane K0 + n of
// the group, through the DPP row of bx, by) in the lanes i <= J and i >= k.
// NOP: a leading s_nop for the DPP reads, where a block label may precede.
#define EQ_COL_EXEC(M) "s_mov_b32 exec_lo, " M "\n\ts_mov_b32 exec_hi, " M "\n\t"
#define EQ_COL_FMAC(X, Y, BX, BY, SX, SY, K)                                                      \
  "v_fmac_f32_dpp " X ", -" BX ", " SX " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n\t"       \
  "v_fmac_f32_dpp " Y ", -" BX ", " SY " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n\t"       \
  "v_fmac_f32_dpp " X ", -" BY ", " SY " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n\t"       \
  "v_fmac_f32_dpp " Y ", " BY ", " SX " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n\t"
#define EQ_COL_TAIL "s_mov_b64 exec, -1"
template <int UT, int J, int K0, int N, bool NOP>
__device__ __forceinline__ void elim_cols(float2 *v, float bx, float by, float2 s) {
  constexpr uint32_t le = ~lanes_ge<UT>(J + 1);
  constexpr int m0 = (int)(le | lanes_ge<UT>(K0)), m1 = (int)(le | lanes_ge<UT>(K0 + 1));
  constexpr int m2 = (int)(le | lanes_ge<UT>(K0 + 2)), m3 = (int)(le | lanes_ge<UT>(K0 + 3));
  constexpr int k0 = K0 % 16;
  if constexpr (NOP) asm volatile("s_nop 2");  // and the two scalar moves
  if constexpr (N == 4) {
    asm volatile(EQ_COL_EXEC("%12") EQ_COL_FMAC("%0", "%1", "%8", "%9", "%10", "%11", "%16")
                     EQ_COL_EXEC("%13") EQ_COL_FMAC("%2", "%3", "%8", "%9", "%10", "%11", "%17")
                     EQ_COL_EXEC("%14") EQ_COL_FMAC("%4", "%5", "%8", "%9", "%10", "%11", "%18")
                     EQ_COL_EXEC("%15") EQ_COL_FMAC("%6", "%7", "%8", "%9", "%10", "%11", "%19") EQ_COL_TAIL
                 : "+&v"(v[0].x), "+&v"(v[0].y), "+&v"(v[1].x), "+&v"(v[1].y), "+&v"(v[2].x), "+&v"(v[2].y),
                   "+&v"(v[3].x), "+&v"(v[3].y)
                 : "v"(bx), "v"(by), "v"(s.x), "v"(s.y), "n"(m0), "n"(m1), "n"(m2), "n"(m3), "n"(k0), "n"(k0 + 1),
                   "n"(k0 + 2), "n"(k0 + 3));
  } else if constexpr (N == 3) {
    asm volatile(EQ_COL_EXEC("%10") EQ_COL_FMAC("%0", "%1", "%6", "%7", "%8", "%9", "%13")
                     EQ_COL_EXEC("%11") EQ_COL_FMAC("%2", "%3", "%6", "%7", "%8", "%9", "%14")
                     EQ_COL_EXEC("%12") EQ_COL_FMAC("%4", "%5", "%6", "%7", "%8", "%9", "%15") EQ_COL_TAIL
                 : "+&v"(v[0].x), "+&v"(v[0].y), "+&v"(v[1].x), "+&v"(v[1].y), "+&v"(v[2].x), "+&v"(v[2].y)
                 : "v"(bx), "v"(by), "v"(s.x), "v"(s.y), "n"(m0), "n"(m1), "n"(m2), "n"(k0), "n"(k0 + 1),
                   "n"(k0 + 2));
  } else if constexpr (N == 2) {
    asm volatile(EQ_COL_EXEC("%8") EQ_COL_FMAC("%0", "%1", "%4", "%5", "%6", "%7", "%10")
                     EQ_COL_EXEC("%9") EQ_COL_FMAC("%2", "%3", "%4", "%5", "%6", "%7", "%11") EQ_COL_TAIL
                 : "+&v"(v[0].x), "+&v"(v[0].y), "+&v"(v[1].x), "+&v"(v[1].y)
                 : "v"(bx), "v"(by), "v"(s.x), "v"(s.y), "n"(m0), "n"(m1), "n"(k0), "n"(k0 + 1));
  } else if constexpr (N == 1) {
    asm volatile(EQ_COL_EXEC("%6") EQ_COL_FMAC("%0", "%1", "%2", "%3", "%4", "%5", "%7") EQ_COL_TAIL
                 : "+&v"(v[0].x), "+&v"(v[0].y)
                 : "v"(bx), "v"(by), "v"(s.x), "v"(s.y), "n"(m0), "n"(k0));
  }
}
#undef EQ_COL_EXEC
#undef EQ_COL_FMAC
#undef EQ_COL_TAIL

// What the elimination carries besides the matrix rows.  npos counts, per
// group (one 64 / NSYS-bit field each, scalar arithmetic), the leading
// pivots that were positive; okm masks the groups whose pivots all were.
struct Elim {
  float2 acc;  // t of the lanes ahead, -z of the lanes done
  float d;     // [A^{-1}]_uu of the lanes done
  uint64_t okm, npos;
};

// Step J.  ZERO: v[J] is left as conj(X_Ju) in lane u (zero in lanes past J
// of the same 16 rows), for callers that use X.
template <int UT, int J, bool ZERO, bool RHS>
__device__ __forceinline__ void elim_step(float2 (&v)[16], Elim &e, float rho, int U) {
  constexpr int j = J % 16, P = J - j;
  // the shift of A = G + rho I enters here: nothing else reads the diagonal
  const float ajj = gbcast<UT, J>(v[j].x) + rho;
  e.okm &= __ballot(ajj > 0.f);
  e.npos += e.okm & (UT == 16 ? 0x0001000100010001ull : 0x0000000100000001ull);
  // hardware reciprocal square root (about 1 ulp): 1 / L_JJ
  const float inv = __builtin_amdgcn_rsqf(ajj);
  const bool me = lanes(lanes_ge<UT>(J) & ~lanes_ge<UT>(J + 1));
  float2 s = make_float2(v[j].x * inv, v[j].y * inv);
  if (me) s = make_float2(inv, 0.f);
  float d = e.d;
  if (me) d = 0.f;
  e.d = d + fmaf(s.x, s.x, s.y * s.y);  // one rounding of the running sum a step
  const BSrc bx = bsrc<UT>(s.x), by = bsrc<UT>(s.y);
  if constexpr (RHS) {
    const BSrc tx = bsrc<UT>(e.acc.x * inv), ty = bsrc<UT>(e.acc.y * inv);
    if (me) e.acc = make_float2(0.f, 0.f);
    // acc -= s t_J, the product rounded before it is subtracted (the running
    // sum is rounded once a step: 5% less error in z than four FMACs on it).
    // The s_nop also covers the columns that follow.
    float px, py;
    asm volatile("s_nop 1\n\t"
                 "v_mul_f32_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                 "v_mul_f32_dpp %1, %2, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %0, -%3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %1, %3, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
                 : "=&v"(px), "=&v"(py)
                 : "v"(bpick<J>(tx)), "v"(bpick<J>(ty)), "v"(s.x), "v"(s.y), "n"(j), "v"(bpick<J>(bx)),
                   "v"(bpick<J>(by)));
    e.acc.x -= px;
    e.acc.y -= py;
  } else {
    asm volatile("s_nop 1" : : "v"(bpick<J>(bx)), "v"(bpick<J>(by)));
  }
  sfor<4>([&](auto G) {
    constexpr int g = G;
    constexpr int k0 = j + 1 > 4 * g ? j + 1 : 4 * g, n = 4 * g + 4 - k0;
    if constexpr (n > 0) {
      // columns of padded users only: nothing to update
      if (g == j / 4 || U > P + 4 * g) elim_cols<UT, J, P + k0, n, g != j / 4>(&v[k0], bpick<J>(bx), bpick<J>(by), s);
    }
  });
  if constexpr (ZERO) {
    constexpr uint32_t end = UT == 32 && P == 0 ? lanes_ge<UT>(16) : 0u;
    v[j] = lanes(lanes_ge<UT>(J + 1) & ~end) ? make_float2(0.f, 0.f) : s;
  }
  step_fence();
}

// Steps J .. END-1 of those below U (wave-uniform).  The steps of padded users
// are left out, so nothing reads their rows and columns.
template <int UT, int J, int END, bool ZERO, bool RHS>
__device__ __forceinline__ void elim_steps(float2 (&v)[16], Elim &e, float rho, int U) {
  elim_step<UT, J, ZERO, RHS>(v, e, rho, U);
  if constexpr (J + 1 < END) {
    if (U > J + 1) elim_steps<UT, J + 1, END, ZERO, RHS>(v, e, rho, U);
  }
}

// Between the halves of a 32 x 32 elimination: with A = [A11 .; A21 A22] in
// 16 x 16 blocks, S = A22 - L21 L21^H and conj(Y) = -conj(L21 X11) for the
// NS systems of the wave, complex products on 16x16x4 FP32 MFMA (four real
// products each).  The slot of a system holds conj(X11) (row u: column u) in
// its block 0, L21 in block 1 and A22 in block 2; S replaces A22 and conj(Y)
// (row u: column u) replaces L21.
template <int NS>
__device__ __forceinline__ void elim_middle(float2 *A) {
  const int lane = lane_id();
  const int lr = lane % 16, lg = lane / 16;
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    float2 *As = A + q * kSlot<32>;
    f4 sr, si, yr, yi;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float2 a22 = blk_el(As, 2, 4 * lg + r, lr);
      sr[r] = a22.x;
      si[r] = a22.y;
      yr[r] = 0.f;
      yi[r] = 0.f;
    }
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) {
      const float2 l = blk_el(As, 1, lr, 4 * kc + lg);  // L21[lr][k]
      const float2 x = blk_el(As, 0, lr, 4 * kc + lg);  // conj(X11)[k][lr]
      // S -= l conj(l'),  conj(Y) -= conj(l) conj(x)
      sr = mma32(-l.x, l.x, sr);
      yr = mma32(-l.x, x.x, yr);
      si = mma32(l.x, l.y, si);
      yi = mma32(-l.x, x.y, yi);
      sr = mma32(-l.y, l.y, sr);
      yr = mma32(-l.y, x.y, yr);
      si = mma32(-l.y, l.x, si);
      yi = mma32(l.y, x.x, yi);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      blk_el(As, 2, 4 * lg + r, lr) = make_float2(sr[r], si[r]);
      blk_el(As, 1, lr, 4 * lg + r) = make_float2(yr[r], yi[r]);
    }
  }
}

template <int UT>
struct LocalSolve {
  float2 z;     // [(G + rho I)^{-1} m]_u
  float d;      // [(G + rho I)^{-1}]_uu
  float norm1;  // bound of ||G + rho I||_1
  int fail;     // 0, or the first pivot that is not positive, + 1
  bool bad;     // a non-finite entry in G or m
};

// Solves (G + rho I) z = m for the system of each lane group, G in the
// group's packed slot (of NS slots from A; entries of padded users zero).
// Lane i is user i; rho may differ between the groups.  KEEP: conj(X), X =
// L^{-1}, is left in the slot: row u of blocks 0 and 1 (u < 16), or of block
// 2, holds the rows 0..15 and 16..31 of column u (columns of padded users
// are zero).
// Without RHS, m and z are not used.
template <int UT, bool KEEP, int NS, bool RHS = true>
__device__ __forceinline__ void solve_slot(LocalSolve<UT> &r, float2 *A, int slot, int i, float2 m, float rho, int U) {
  U = __builtin_amdgcn_readfirstlane(U);
  float2 *As = A + slot * kSlot<UT>;
  const int h = UT == 32 ? i >> 4 : 0, ii = i & 15;
  float2 v[16];
  float rowsum = 0.f;
  sfor<16>([&](auto K) {
    constexpr int k = K;
    const float2 a = blk_el(As, h, ii, k);
    rowsum = abs_row_acc(rowsum, a);
    v[k] = lanes(lanes_ge<UT>(k)) ? a : make_float2(0.f, 0.f);
  });
  if constexpr (UT == 32) {
    // the rest of the row, for the norm (column ii of block 1 is its
    // conjugate in the rows 0..15); A22 stays in the slot
    sfor<16>([&](auto K) {
      constexpr int k = K;
      rowsum = abs_row_acc(rowsum, As[256 * (1 + h) + (h ? 16 * ii + (k ^ ii) : 16 * k + (ii ^ k))]);
    });
  }
  r.bad = gany<UT>(!isfinite(abs_row_acc(rowsum, m)));
  r.norm1 = gmax<UT>(i < U ? fmaf(rowsum, 1.f / kRowScale, rho) : 0.f);
  Elim e;
  e.acc = m;
  e.d = 0.f;
  e.okm = ~0ull;
  e.npos = 0;
  elim_steps<UT, 0, 16, KEEP || UT == 32, RHS>(v, e, rho, U);
  if constexpr (UT == 32) {
    // conj(X11) by columns from the first 16 lanes, L21 by rows from the others
    sfor<16>([&](auto K) {
      constexpr int k = K;
      blk_el(As, h, ii, k) = v[k];
    });
    wave_sync();
    elim_middle<NS>(A);
    wave_sync();
    sfor<16>([&](auto K) {
      constexpr int k = K;
      const float2 a = blk_el(As, 1 + h, ii, k);
      v[k] = lanes(lanes_ge<UT>(16 + k) | ~lanes_ge<UT>(16)) ? a : make_float2(0.f, 0.f);
    });
    elim_steps<UT, 16, 32, KEEP, RHS>(v, e, rho, U);
  }
  if constexpr (KEEP) {
    sfor<16>([&](auto K) {
      constexpr int k = K;
      blk_el(As, UT == 32 ? 1 + h : 0, ii, k) = v[k];
    });
  }
  r.z = make_float2(-e.acc.x, -e.acc.y);
  r.d = e.d;
  const int npos = UT == 16 ? (int)(e.npos >> (16 * (lane_id() / 16))) & 0xffff : (int)(e.npos >> (32 * (lane_id() / 32)));
  r.fail = npos == U ? 0 : npos + 1;
}

// Unbiased L-MMSE: the L-MMSE estimate of user u has gain
// mu_u = [(G + rho I)^{-1} G]_uu = 1 - rho d_u = 1 - sigma2_u / E_s; returns
// 1 / mu_u for ub = 1/E_s, and exactly 1 for ub = 0 (biased L-MMSE, ZF).
__device__ __forceinline__ float unbias_factor(float s2, float ub) { return 1.0f / (1.0f - s2 * ub); }

}  // namespace dbpeq
