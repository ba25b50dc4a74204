// Forward kernels: fused Gram + matched filter + fusion + L-MMSE solve.
//
// PD (Section II-C, Section III-A): a wave equalises NSYS subcarriers.  The
// adder tree of eq. (fullMRC) is the MFMA accumulator itself: the row blocks
// of all clusters are accumulated into one G and one y^MRC, so the per-cluster
// statistics are summed on chip and never leave the wave.
//
// FD (Section II-D, Section IV): a wave equalises all clusters of `spw`
// subcarriers, or up to four waves share those of one, NSYS local systems per
// round; after each round the lane groups' estimates and variances are summed
// across the wave in registers, with the weights of Lemma 1 (eq. (opt_fusion)),
// into the fusion sums of eq. (fusionrule), which the waves of a subcarrier
// exchange once, through LDS.
//
// The precision forms differ only in the Gram product (FP32 MFMA, BF16 MFMA,
// or three BF16 MFMA products of split operands) and, for the BF16 forms, one
// refinement step z += A^{-1} (H^H (y - H z) - rho z) with the FP32 residual.
// Systems whose condition estimate ||A||_1 * trace(A^{-1}) exceeds
// EQ_COND_LIMIT, or whose pivot failed, are queued for an FP64 re-solve.
#include "eq_round.h"

#ifndef EQ_WAVES_PER_EU
#define EQ_WAVES_PER_EU 4
#endif
#ifndef EQ_PD_PER32
#define EQ_PD_PER32 1
#endif

namespace dbpeq {

// Queue subcarrier w for the FP64 re-solve (one lane calls this).
__device__ __forceinline__ void enqueue_fp64(const FwdArgs &a, int w) {
  const int pos = atomicAdd(a.fb_count, 1);
  if (pos >= 0 && pos < a.W) a.fb_list[pos] = w;  // capacity W
}

// Most PD systems per work item.  A 32-lane group streams 32 KiB..1 MiB per
// system, so one system per item keeps the work items short enough to fill
// the device several times over (two per item left most of it idle during
// the last generation of workgroups).
template <int UT, int PREC>
constexpr int pd_per() {
  return UT == 32 ? EQ_PD_PER32 : (refines(PREC) ? 2 : 64 / UT);
}

// Occupancy target, waves per SIMD.  UT = 16: 4 (128 VGPRs; FD takes 108, and
// 124 with the split-BF16 Gram, without spills), 3 (168) for the refining forms,
// which hold the solution across the residual pass.  UT = 32: 4 for PD, 3 for FD
// (156; 168 with the split-BF16 Gram, which spills 76 bytes), 2 for the refining
// forms.
template <int UT, int PREC, bool FD>
constexpr int waves_target() {
  if (UT == 32) return refines(PREC) ? 2 : (FD ? 3 : 4);
  return refines(PREC) ? 3 : EQ_WAVES_PER_EU;
}

template <int UT, int PREC, class SM>
__device__ __forceinline__ void pd_task(const FwdArgs &a, int w0, int nvalid, SM &sm) {
  const int lane = lane_id();
  const int sme = lane / UT;
  const int i = lane % UT;
  const size_t HB = (size_t)a.B * a.U;
  auto seg = [&](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
    const size_t w = (size_t)w0 + s;
    Hw = a.H + w * HB;
    yw = a.y + w * a.B;
    r0 = 0;
    r1 = a.B;
  };

  // ---- Gram + matched filter of the round's subcarriers (all clusters
  //      accumulate into one G and one y^MRC: the adder tree of eq. (fullMRC))
  gram_stream<UT, PREC, refines(PREC) ? kLoadKeep : kLoadLast>(nvalid, a.U, seg, [&](int s, const Acc<UT> &acc, float2 mf) {
    store_gram_packed<UT, PREC>(gram_addr<UT>(), sm.A + s * kSlot<UT>, acc);
    sm.M[s][lane] = mf;
  });
  wave_sync();

  // ---- factor and solve: group sme, row/column i (the groups past the last
  //      system solve what is in their slot, and write nothing)
  const int w = w0 + sme;
  const bool live = sme < nvalid;
  LocalSolve<UT> r;
  local_solve<UT, refines(PREC)>(r, sm, slot_of<SM>(sme), i, a.rho, a.U);
  if constexpr (refines(PREC)) refine_round<UT>(r, sm, nvalid, a.U, [&](int) { return a.rho; }, seg, live);

  const float kappa = r.norm1 * gsum<UT>(i < a.U ? r.d : 0.f);
  const bool routed = live && !r.bad && (r.fail != 0 || !(kappa <= EQ_COND_LIMIT));
  if (live) {
    if (i < a.U) {
      const float nanv = __int_as_float(0x7fc00000);
      const float s2 = a.n0 * r.d, k = a.ub != 0.f ? unbias_factor(s2, a.ub) : 1.f;
      a.z[(size_t)w * a.U + i] = r.bad ? make_float2(nanv, nanv) : make_float2(r.z.x * k, r.z.y * k);
      if (a.s2) a.s2[(size_t)w * a.U + i] = r.bad ? nanv : s2 * k;
    }
    if (i == 0) {
      if (a.info) a.info[w] = (r.bad ? -1 : r.fail) | (routed ? EQ_INFO_FP64 : 0);
      if (routed) enqueue_fp64(a, w);
    }
  }
}

// All clusters of subcarriers w0 .. w0+nsub-1, NSYS clusters per round.  The
// nw waves of the workgroup take the rounds in turn (nsub = 1 if nw > 1);
// sms: the LDS of all of them.
template <int UT, int PREC, class SM>
__device__ __forceinline__ void fd_task(const FwdArgs &a, int w0, int nsub, SM *sms, int wv, int nw) {
  constexpr int NSYS = 64 / UT;
  SM &sm = sms[wv];
  const int lane = lane_id();
  const int sme = lane / UT;
  const int i = lane % UT;
  const size_t HB = (size_t)a.B * a.U;
  const int C = a.C;
  // clusters of the subcarriers of this task
  const int ntot = nsub * C;
  const bool user_nu = a.nu != nullptr;
  const float nanv = __int_as_float(0x7fc00000);
  // lane groups per subcarrier of a round (C is 1 or 2 when it holds several)
  const int gw = a.spw > 1 ? C : NSYS;

  // fusion sums of user i of the group's subcarrier, and the lanes whose
  // cluster was routed to FP64
  float sw = 0.f, szx = 0.f, szy = 0.f;
  unsigned long long routedm = 0;

  const GramAddr<UT> ga = gram_addr<UT>();
  for (int base = wv * NSYS; base < ntot; base += nw * NSYS) {
    const int nvalid = min(NSYS, ntot - base);
    auto seg = [&](int s, const float2 *&Hw, const float2 *&yw, int &r0, int &r1) {
      const int idx = base + s;
      const int wl = idx / C, c = idx - wl * C;
      const size_t w = (size_t)(w0 + wl);
      Hw = a.H + w * HB;
      yw = a.y + w * a.B;
      cluster_rows<FwdArgs>(c, r0, r1);
    };
    // ---- local Gram + MRC of the clusters of this round
    gram_stream<UT, PREC, refines(PREC) ? kLoadKeep : kLoadLast>(nvalid, a.U, seg, [&](int s, const Acc<UT> &acc, float2 mf) {
      store_gram_packed<UT, PREC>(ga, sm.A + s * kSlot<UT>, acc);
      sm.M[s][lane] = mf;
    });
    wave_sync();

    // ---- local L-MMSE of cluster (wl, c) by group sme
    const int idx = base + sme;
    const int wl = idx / C, c = idx - wl * C;
    const int w = w0 + wl;
    const bool live = sme < nvalid;
    LocalSolve<UT> r;
    local_solve<UT, refines(PREC)>(r, sm, sme, i, a.rho, a.U);
    if constexpr (refines(PREC)) refine_round<UT>(r, sm, nvalid, a.U, [&](int) { return a.rho; }, seg, live);

    const float kappa = r.norm1 * gsum<UT>(i < a.U ? r.d : 0.f);
    const bool routed = live && !r.bad && (r.fail != 0 || !(kappa <= EQ_COND_LIMIT));
    if (live && i == 0 && a.info) a.info[(size_t)w * C + c] = (r.bad ? -1 : r.fail) | (routed ? EQ_INFO_FP64 : 0);
    routedm |= __ballot(routed);
    // ---- fusion terms of this cluster: its weight times the local estimate,
    //      and the weight (optimal: 1 / sigma2_c) or nu^2 sigma2_c (given
    //      weights); estimate and variance are scaled to unit gain for the
    //      unbiased L-MMSE
    const float k = a.ub != 0.f ? unbias_factor(a.n0 * r.d, a.ub) : 1.f;
    const float s2c = a.n0 * r.d * k;
    float p, q;
    if (user_nu) {
      p = live && i < a.U ? a.nu[((size_t)w * C + c) * a.U + i] : 0.f;
      q = p * p * s2c;
    } else {
      p = q = 1.0f / s2c;
    }
    const float pk = p * k;
    float fx = r.bad ? nanv : pk * r.z.x, fy = r.bad ? nanv : pk * r.z.y;
    if (r.bad) q = nanv;
    if (!live) fx = fy = q = 0.f;
    szx += group_sum<UT>(fx, gw);
    szy += group_sum<UT>(fy, gw);
    sw += group_sum<UT>(q, gw);
    wave_sync();
  }

  if (nw > 1) {
    // the waves' sums meet in wave order
    float *part = &sm.M[0][0].x;
    if (lane < UT) {
      part[lane] = szx;
      part[UT + lane] = szy;
      part[2 * UT + lane] = sw;
    }
    if (lane == 0) part[3 * UT] = routedm != 0 ? 1.f : 0.f;
    __syncthreads();
    if (wv != 0) return;
    szx = szy = sw = 0.f;
    for (int q = 0; q < nw; ++q) {
      const float *o = &sms[q].M[0][0].x;
      szx += o[i];
      szy += o[UT + i];
      sw += o[2 * UT + i];
      if (o[3 * UT] != 0.f) routedm = ~0ull;
    }
  }
  const int wl = sme / gw;
  if (sme == wl * gw && wl < nsub) {
    const int w = w0 + wl;
    if (i < a.U) {
      const float inv = 1.0f / sw;
      a.z[(size_t)w * a.U + i] = user_nu ? make_float2(szx, szy) : make_float2(szx * inv, szy * inv);
      if (a.s2) a.s2[(size_t)w * a.U + i] = user_nu ? sw : inv;
    }
    const unsigned long long mine = (gw * UT == 64 ? ~0ull : (1ull << (gw * UT)) - 1ull) << (sme * UT);
    if (i == 0 && (routedm & mine)) enqueue_fp64(a, w);
  }
}

// PD: one wave per workgroup; workgroup b takes systems b spw .. of W.
template <int UT, int PREC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(waves_target<UT, PREC, false>(), 8))) void eq_forward_pd_kernel(const FwdArgs a) {
  constexpr int per = pd_per<UT, PREC>();
  // work items of fewer systems than lane groups need fewer matrix slots
  __shared__ SolveSmem<UT, refines(PREC), (per < 64 / UT ? per : 64 / UT)> sm;
  const int w0 = blockIdx.x * a.spw;
  pd_task<UT, PREC>(a, w0, min(a.spw, a.W - w0), sm);
}

// FD: blockDim / 64 waves per workgroup (fd_waves), `spw` subcarriers.
constexpr int kFdWaves = 4;
template <int UT, int PREC>
__global__ __launch_bounds__(64 * kFdWaves) __attribute__((amdgpu_waves_per_eu(waves_target<UT, PREC, true>(), 8))) void eq_forward_fd_kernel(const FwdArgs a) {
  extern __shared__ __align__(128) float2 fd_lds[];
  using SM = SolveSmem<UT, refines(PREC)>;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), nw = blockDim.x / 64;
  const int w0 = blockIdx.x * a.spw;
  fd_task<UT, PREC>(a, w0, min(a.spw, a.W - w0), reinterpret_cast<SM *>(fd_lds), wv, nw);
}

__global__ void zero_i32_kernel(int32_t *p, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) p[t] = 0;
}

hipError_t launch_zero_i32(int32_t *p, int n, hipStream_t s) {
  hipLaunchKernelGGL(zero_i32_kernel, dim3((n + 63) / 64), dim3(64), 0, s, p, n);
  return hipGetLastError();
}

// Waves per FD workgroup: one per round of a subcarrier, at most kFdWaves.  A
// subcarrier of B = 1024, C = 16, U = 32 keeps one wave busy for about 0.2 ms
// and 4,800 of them were barely more than two generations of one-wave
// workgroups: 490 us with one wave each, 458 with two, 428 with four (the
// 38,400 subcarriers of B = 256, C = 8, U = 16 take 317 us either way, the
// 1,200 of one symbol 26.6 against 23.8 us).
static int fd_waves(int UT, int C) {
  const int rounds = (C * UT + 63) / 64;
  return rounds < kFdWaves ? rounds : kFdWaves;
}

template <int UT, int PREC, bool FD>
static hipError_t launch_one(const FwdArgs &a, hipStream_t s) {
  // one work item per workgroup: the hardware dispatcher refills a freed slot
  // at once (a one-generation grid with equal shares per workgroup measured
  // slower: its partial rounds add solves)
  if constexpr (FD) {
    const int nw = a.spw > 1 ? 1 : waves_in_launch(a.W, fd_waves(UT, a.C));
    hipLaunchKernelGGL((eq_forward_fd_kernel<UT, PREC>), dim3((a.W + a.spw - 1) / a.spw), dim3(64 * nw),
                       nw * sizeof(SolveSmem<UT, refines(PREC)>), s, a);
  } else {
    FwdArgs b = a;
    b.spw = pd_share(a.W, pd_per<UT, PREC>());
    hipLaunchKernelGGL((eq_forward_pd_kernel<UT, PREC>), dim3((a.W + b.spw - 1) / b.spw), dim3(64), 0, s, b);
  }
  return hipGetLastError();
}

template <int UT, bool FD>
static hipError_t launch_prec(const FwdArgs &a, int prec, hipStream_t s) {
  switch (prec) {
    case PREC_FP32: return launch_one<UT, PREC_FP32, FD>(a, s);
    case PREC_BF16:  // PD only (eq_fd refuses the single-BF16 Gram)
      if constexpr (FD) return hipErrorInvalidValue;
      else return launch_one<UT, PREC_BF16, FD>(a, s);
    case PREC_BF16X3: return launch_one<UT, PREC_BF16X3, FD>(a, s);
    default: return launch_one<UT, PREC_BF16X3_NR, FD>(a, s);
  }
}

hipError_t launch_forward(const FwdArgs &a, bool fd, int prec, hipStream_t s) {
  const int UT = ut_for(a.U);
  if (UT == 16) return fd ? launch_prec<16, true>(a, prec, s) : launch_prec<16, false>(a, prec, s);
  return fd ? launch_prec<32, true>(a, prec, s) : launch_prec<32, false>(a, prec, s);
}

}  // namespace dbpeq
