// The gradient walks of the one-direction loss (grad_walk.h), and the launcher of the gradient pass of every bf16 MFMA call.
#include "grad_walk.h"

namespace gc {

template <int D>
__global__ void __launch_bounds__(256) GR_CODE_ALIGN grad_mfma_kernel(GradArgs ga) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gsmem[];
  check_shared_positives(ga);
  const int nQ = ga.obQ * ga.nsq;
  const int id = xcd_task_id();
  if (id < nQ) {
    grad_body<D, true, false>(ga, id % ga.obQ, id / ga.obQ, gsmem);
  } else {
    const int t = id - nQ;
    grad_body<D, false, false>(ga, t % ga.obP, t / ga.obP, gsmem);
  }
}

// the online-statistics walk: every workgroup has the dQ role
template <int D>
__global__ void __launch_bounds__(256) GR_CODE_ALIGN grad_online_kernel(GradArgs ga) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gsmem[];
  const int id = xcd_task_id();
  grad_body<D, true, false, true>(ga, id % ga.obQ, id / ga.obQ, gsmem);
}
template <int D>
static hipError_t grad_online_launch(const GradArgs& ga, int nwg, hipStream_t stream) {
  const int smem = GradCfg<D>::SMEM;
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)grad_online_kernel<D>, smem, attr_done); e != hipSuccess) return e;
  grad_online_kernel<D><<<nwg, 256, smem, stream>>>(ga);
  return hipGetLastError();
}

// dQ partials (scaled by alpha / B, relative to each split's reference) and the statistics of every split
hipError_t launch_grad_online(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  GradArgs ga{};
  ga.Q = (const unsigned short*)a.q; ga.P = (const unsigned short*)a.p;
  ga.pos_pad = a.pos_idx; ga.lse2 = nullptr; ga.lse2_t = nullptr;
  ga.B = a.B; ga.Pn = a.P;
  ga.alpha2 = a.alpha * kLog2e; ga.out_scale = a.alpha / (float)a.B * (a.grad_mul != 0.f ? a.grad_mul : 1.f);
  ga.mask_self = (a.flags & GC_MASK_SELF) ? 1 : 0;
  ga.obQ = (a.B + GR_OWN - 1) / GR_OWN; ga.nsq = pl.fz_nsq; ga.q_stream_len = pl.fz_q_stream_len;
  ga.dq_out = (float*)(ws + pl.off_dq_part); ga.dq_split_stride = (size_t)a.B * a.d;
  ga.on_ref = (float*)(ws + pl.off_on_ref); ga.on_best = (float*)(ws + pl.off_part_m); ga.on_l = (float*)(ws + pl.off_part_l);
  ga.on_idx = (int*)(ws + pl.off_part_idx); ga.on_pos = (float*)(ws + pl.off_pos);
  ga.on_argmax = a.argmax ? 1 : 0;
  const int nwg = ga.obQ * ga.nsq;
  switch (a.d) {
    case 256: return grad_online_launch<256>(ga, nwg, a.stream);
    case 384: return grad_online_launch<384>(ga, nwg, a.stream);
    case 512: return grad_online_launch<512>(ga, nwg, a.stream);
    case 640: return grad_online_launch<640>(ga, nwg, a.stream);
    case 768: return grad_online_launch<768>(ga, nwg, a.stream);
    default: return hipErrorInvalidValue;
  }
}

template <int D>
static hipError_t grad_mfma_launch(const GradArgs& ga, int nwg, hipStream_t stream) {
  const int smem = GradCfg<D>::SMEM;
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)grad_mfma_kernel<D>, smem, attr_done); e != hipSuccess) return e;
  grad_mfma_kernel<D><<<nwg, 256, smem, stream>>>(ga);
  return hipGetLastError();
}
hipError_t launch_grad_mfma(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  GradArgs ga{};
  ga.Q = (const unsigned short*)a.q; ga.P = (const unsigned short*)a.p;
  ga.pos_pad = (const int32_t*)(ws + pl.off_pos_pad); ga.lse2 = (const float*)(ws + pl.off_lse2);
  ga.lse2_t = a.lse2_t;
  ga.B = a.B; ga.Pn = a.P;
  ga.alpha2 = a.alpha * kLog2e; ga.out_scale = a.alpha / (float)a.B * (a.grad_mul != 0.f ? a.grad_mul : 1.f);
  ga.mask_self = (a.flags & GC_MASK_SELF) ? 1 : 0;
  // NT-Xent in one walk: q = p = z, so the score matrix is symmetric, target j's log-sum-exp is anchor j's, and
  //   dz_i = (alpha/n) sum_j (g_ij + g_ji) z_j,   g_ij + g_ji = 2^(t_ij - lse2_i) + 2^(t_ij - lse2_j) - 2 [j = pair(i)]:
  // twice the coefficient of the symmetric loss with both statistics taken from the one array.  Only the dQ role runs.
  const bool one_walk = pl.one_walk && a.dz;
  ga.wexp = a.wexp; ga.wexp_t = a.wexp_t; ga.wide = a.wide;
  if (one_walk) { ga.lse2_t = ga.lse2; ga.wexp_t = ga.wexp; ga.out_scale *= 2.f; }
  const bool want_q = a.dq || a.dz, want_p = (a.dp || a.dz) && !one_walk;
  const size_t nq = (size_t)a.B * a.d, np = (size_t)a.P * a.d;
  const bool few = few_kernel(a, pl);
  const int own = few ? kFewOwn : (a.d == 128) ? G1_OWN : GR_OWN;   // owner rows per workgroup
  ga.obQ = want_q ? (a.B + own - 1) / own : 0; ga.nsq = pl.nsq; ga.q_stream_len = pl.q_stream_len;
  ga.obP = want_p ? (a.P + own - 1) / own : 0; ga.nsp = pl.nsp; ga.p_stream_len = pl.p_stream_len;
  // every output goes through the kernel that sums the split partials (a single split included): it adds the
  // positive's term in fp32 (PosFix) and rounds a bf16 cache
  const bool cache_bf16 = (a.flags & GC_CACHE_BF16) != 0;
  ga.dq_out = (float*)(ws + pl.off_dq_part); ga.dq_split_stride = nq;
  ga.dp_out = (float*)(ws + pl.off_dp_part); ga.dp_split_stride = np;
  // the symmetric loss inverts its pairing itself (a bijection); one direction: the merge left an anchor per target
  const bool sym_pairs = a.lse2_t != nullptr;
  if (want_p && !sym_pairs) { ga.inv = (const int32_t*)(ws + pl.off_inv); ga.shared = (int*)(ws + pl.off_err) + 1; }
  const int nwg = ga.obQ * ga.nsq + ga.obP * ga.nsp;
  if (nwg == 0) { prof_mark_grad_kernel_done(a.stream); return hipSuccess; }
  hipError_t e;
  FewMerge fm{};
  if (merges_itself(a, pl)) {
    ga.pos_pad = a.pos_idx;
    fm = few_merge_args(a, pl);
  }
  if (few) e = grad_few_launch(ga, fm, a.d, nwg, a.stream);
  else if (a.d == 128) e = grad128_launch(ga, nwg, a.stream);
  else if (ga.lse2_t) e = grad_sym_launch(ga, a.d, nwg, a.stream);
  else switch (a.d) {
    case 256: e = grad_mfma_launch<256>(ga, nwg, a.stream); break;
    case 384: e = grad_mfma_launch<384>(ga, nwg, a.stream); break;
    case 512: e = grad_mfma_launch<512>(ga, nwg, a.stream); break;
    case 640: e = grad_mfma_launch<640>(ga, nwg, a.stream); break;
    case 768: e = grad_mfma_launch<768>(ga, nwg, a.stream); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  prof_mark_grad_kernel_done(a.stream);
  // fixed-order sums of the split partials, each with the positive's term of its rows: one launch, which also sums the
  // row losses if asked to
  PosFix fx{};
  fx.pos = ga.pos_pad; fx.pos_t = (const float*)(ws + pl.off_pos); fx.lse2 = ga.lse2; fx.lse2_t = ga.lse2_t;
  fx.B = a.B; fx.P = a.P; fx.d = a.d; fx.scale = ga.out_scale;
  ReduceJob job[2] = {};
  int n = 0;
  if (want_q) {   // rows are anchors (NT-Xent, one walk: the positive of view i is view i ^ 1)
    ReduceJob& j = job[n++];
    j.out = a.dz ? (void*)a.dz : (void*)a.dq; j.n = nq; j.nsrc = 1; j.ptr[0] = ga.dq_out; j.count[0] = pl.nsq; j.stride[0] = nq;
    j.out_bf16 = cache_bf16 && !a.dz;
    j.fix = fx; j.fix.mode = 1; j.fix.other = ga.P;
  }
  if (want_p) {
    ReduceJob& j = job[n++];
    j.out = a.dp; j.n = np; j.nsrc = 1; j.ptr[0] = ga.dp_out; j.count[0] = pl.nsp; j.stride[0] = np;
    j.out_bf16 = cache_bf16;
    j.fix = fx; j.fix.mode = 2; j.fix.other = ga.Q;
    j.fix.inv = sym_pairs ? a.pos_inv : ga.inv; j.fix.shared = sym_pairs ? a.zero_word : ga.shared;
  }
  return launch_reduce_jobs(job, n, a.stream, a.loss_with_partials ? &a : nullptr, &pl);
}

}  // namespace gc
