// Shared host/device declarations of the gfx950 Gradient Cache library
// (internal; the public C ABI is include/gradcache.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "gradcache.h"

namespace gc {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kNumCUDefault = 256;  // MI355X; what num_cu() answers when no device can be asked
int num_cu();                       // compute units of the current device: sizes grids and workspace splits

// fp32 -> bf16 bits, round to nearest even (inputs here are finite).
__device__ __forceinline__ unsigned short f2bf(float f) {
  unsigned u = __builtin_bit_cast(unsigned, f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short b) { return __builtin_bit_cast(float, (unsigned)b << 16); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// ---------------------------------------------------------------------------
// Workspace plan of gc_loss_and_rep_grad_ex: one host function decides the
// splits and the byte offsets, so gc_workspace_bytes and the launch agree.
// ---------------------------------------------------------------------------
enum LossRoute {
  ROUTE_MFMA = 0,     // loss_mfma.hip: bf16, d a multiple of 128 up to 768
  ROUTE_PLANES = 1,   // loss_planes.hip: fp32 storage, and bf16 of any other width
  ROUTE_GENERAL = 2,  // loss_generic.hip: the same calls where the workspace is limited and the planes do not fit
  ROUTE_TINY = 3      // loss_generic.hip: the same calls with a handful of scores, in one launch of one workgroup
};
struct LossPlan {
  int route;
  int use_mfma;          // route == ROUTE_MFMA
  int few_grad, few_merge;   // the gradient kernel for short walks (loss_few.hip); it can merge the statistics it needs
  int few_not_q, few_not_p;  // ... but not for the dQ (dP) role alone, see few_kernel
  int one_walk;          // NT-Xent on the MFMA kernels: dz from a single walk (no dP role, no dP partials)
  int stat_splits;       // column (target) ranges of the statistics pass
  int stat_cols_per_split;
  int stat_tile;         // the kernel for few scores (kStatTile); 0: ROUTE_MFMA the 128 x 128 (d = 128: 256-anchor) kernels, ROUTE_PLANES the larger one
  int nsq, nsp;          // stream splits of the dQ-role / dP-role workgroups of the gradient pass
  int q_stream_len, p_stream_len;  // stream rows per split (multiple of the stream tile)
  int b_pad;             // B rounded up to 64 (ROUTE_PLANES: 128): length of the padded lse2 / pos_pad arrays
  // fused mode (MFMA kernels, d >= 256, dQ wanted): no statistics pass; an online-statistics dQ walk, a kernel that
  // merges its splits into lse2 and dQ, then the dP walk.  Each walk fills the GPU alone, so they have splits of their own
  int fused, fused_auto, fz_nsq, fz_nsp, fz_q_stream_len, fz_p_stream_len;   // can run / is chosen without a flag
  // ROUTE_PLANES: bf16 planes per stored value; fragments along d (k-steps of 16, column tiles of 32); rows padded to 128;
  // target tiles per wave of the statistics pass; 32-row blocks a workgroup of the gradient pass owns; column slices;
  // floats between the partials of an output
  int np, px_KS, px_CT, px_rows_q, px_rows_p, px_tiles_per_wave, px_no, px_col_slices, px_ct_per_slice;
  size_t px_stride_q, px_stride_p, off_qk, off_qt, off_pk, off_pt;
  // (everything below off_dq_part is what a call that only forms statistics touches)
  size_t off_err, off_part_m, off_part_l, off_part_idx, off_pos, off_lse2, off_pos_pad, off_rowloss, off_dq_part,
      off_dp_part, off_pos_idx, off_on_ref, off_inv, total;
};

// limit: bytes of workspace there are.  To stay below it the calls of ROUTE_MFMA take fewer splits, those of ROUTE_PLANES
// fewer splits and then ROUTE_GENERAL; what needs the least is returned where nothing fits (the caller compares `total`).
constexpr int kStatTile = 32, kStatBlock = 128;
int stats_block(int B, int P, int d);   // ROUTE_MFMA, d >= 256: edge of a workgroup's scores in the statistics pass, kStatBlock or 256
constexpr int kFewOwn = 32;          // owner rows of a workgroup of the bf16 gradient kernel for few scores (loss_few.hip)
constexpr int kFewMergeRows = 256;   // streamed rows of a workgroup of the gradient kernel for short walks that merges statistics
// ... and rows times splits: every workgroup with the dP role reads so many.  Beyond, a launch that merges them once is faster:
// 512 x 2048 (256 x 64) 2 us, planes of 1024 columns 3.3, 140 x 6000 there (256 x 63) 12; up to it the launch is 1 to 3 us saved.
constexpr int kFewMergeEntries = 160 * 64;
LossPlan make_loss_plan(int B, int P, int d, gc_dtype dt, bool ntxent, size_t limit = (size_t)-1);
void plan_planes(LossPlan& pl, int B, int P, int d, gc_dtype dt, int max_splits);

// Statistics of both sides of a symmetric form from one pass over the scores (stats_mfma_kernel, stats128_both_kernel).
struct LossArgs;
struct BothPlan {
  bool use, triangle;
  int block, n_ablk, cols_per_split, row_slots, nwg;   // owners of a block, blocks; streamed rows of a workgroup; ranges of a block at most
  void partials(const LossArgs& a, const LossPlan& pl, float*& row_m, float*& row_l, float*& col_m, float*& col_l) const;
};
BothPlan plan_both(int n, int d, bool triangle, const LossPlan& pl);

struct LossArgs {
  gc_dtype dt;
  const void* q;
  const void* p;
  const int32_t* pos_idx;
  int B, P, d;
  float alpha;       // scale / temp
  unsigned flags;
  float* loss;
  float* dq;
  float* dp;
  float* lse;
  int32_t* argmax;
  float* dz;         // NT-Xent: dq + dp summed into one buffer (dq, dp then unused)
  float grad_mul;    // extra factor on the gradients (0 = 1; the symmetric loss halves both terms)
  // symmetric loss in one gradient pass (MFMA kernels only): log2-domain log-sum-exp per target over the anchors,
  // padded like the per-anchor one; with it set the statistics of this call are taken as already in `ws`
  const float* lse2_t;
  // ... with the inverse of the pairing (pos_inv[r_i] = i, a bijection there) and a device word that holds 0, for
  // the positive's term of the dP rows (PosFix)
  int32_t* pos_inv;
  const int* zero_word;
  // set by run_loss when the gradient pass ends in a sum of split partials: that launch then also sums the row
  // losses (one launch less); the statistics merge leaves the sum to it
  bool loss_with_partials;
  // symmetric forms: the merge of the statistics also writes 2^(-lse2 - 1) per row (padded with 0), where the partials'
  // indices were (nobody asks these calls for an arg-max), and raises *wide when a row's |lse2| is beyond kWideLse; the
  // gradient pass of the symmetric loss takes both directions' (wexp, wexp_t)
  float* wexp;
  const float* wexp_t;
  int* wide;
  const BothPlan* both;  // the statistics of both sides in one pass; `ws_t`: workspace of the other direction's (symmetric loss)
  char* ws_t;
  const LossArgs* sym[2];   // symmetric loss: the launch that sums its partials also sums the row losses of both directions
  float* sym_loss;
  bool defer_loss_sum;   // the caller sums the row losses itself (the symmetric loss: both directions in one launch)
  char* ws;
  char* ws2;             // base of the offsets from off_dq_part on (ws; the symmetric loss shares that part between its directions)
  hipStream_t stream;
};

// The coefficient of the symmetric forms is 1/2 (2^(t - lse2_i) + 2^(t - lse2_j)) = 2^t (w_i + w_j), w = 2^(-lse2 - 1): one
// exponential a score instead of two, a quarter of the rate each.  With |lse2| up to kWideLse no factor overflows, and
// what 2^t flushes is below 2^(-126 + kWideLse) of its row's sum.  Beyond (one row is enough) the two exponentials stay.
// (d = 128, 16384 views, before that kernel had two waves per SIMD: 233 us with two, 216 with one.)
constexpr float kWideLse = 60.f;

// The positive's own term of Eq. 5 / Eq. 6, (p_{i r_i} - 1) g(t_{r_i}) resp. (p_{i r_i} - 1) f(s_i), is not part of the bf16
// contractions of the MFMA walks (they take the coefficient 0 at the positive): rounded to bf16, this one coefficient
// of size up to 1 next to P - 1 small ones would be the whole error of its gradient row.  The kernel that sums the
// split partials adds it in fp32 from the row statistics:
//   c_i = scale * (2^(pos_t_i - lse2_i) - 1)                                       one direction
//   c_i = scale * (1/2 (2^(pos_t_i - lse2_i) + 2^(pos_t_i - lse2_t[r_i])) - 1)     symmetric loss, NT-Xent
struct PosFix {
  int mode;                     // 0: nothing to add; 1: output rows are anchors (dq, dz); 2: output rows are targets (dp)
  const int32_t* pos;           // [B] r_i
  const int32_t* inv;           // mode 2: [P], inv[j] = an anchor i with r_i = j where there is one (always checked)
  const int* shared;            // mode 2: nonzero when some target is the positive of several anchors (then: a scan)
  const float* pos_t;           // [B] base-2 logit of the positive
  const float* lse2;            // [B] base-2 log-sum-exp per anchor
  const float* lse2_t;          // [P] the same per target over the anchors (symmetric forms), else nullptr
  const unsigned short* other;  // bf16 rows that the term multiplies: targets (mode 1), anchors (mode 2)
  int B, P, d;
  float scale;
};

// The gradient kernel for few scores serves this call.  It owns half as many rows as the long walks: a call for one gradient alone
// that takes it two rounds of workgroups, and them one, is theirs (dp of 100 x 10000 x 512 51.7 us, 45.7 so; dq of 10000 x 100 x 512
// 48.0 and 43.3; not at d = 128: dp of 16 x 20000 33.2 and 35.2).
inline bool few_kernel(const LossArgs& a, const LossPlan& pl) {
  return pl.few_grad && (a.dz || (a.dq ? a.dp || !pl.few_not_q : !pl.few_not_p));
}
// The gradient kernel of this call merges the split statistics: one launch less.  (The dQ role writes what the merge would.)
inline bool merges_itself(const LossArgs& a, const LossPlan& pl) {
  return pl.few_merge && (pl.route != ROUTE_MFMA || few_kernel(a, pl)) && a.dq && !a.lse2_t && !a.wexp && !a.dz;
}

inline void BothPlan::partials(const LossArgs& a, const LossPlan& pl, float*& row_m, float*& row_l, float*& col_m, float*& col_l) const {
  row_m = (float*)(a.ws + pl.off_dq_part);   // (the gradient pass writes there later)
  row_l = row_m + (size_t)row_slots * a.B;
  col_m = row_l + (size_t)row_slots * a.B;
  col_l = col_m + (size_t)n_ablk * a.B;
}

// kernel-launching halves (one per .hip file)
hipError_t launch_stats_both(const LossArgs& a, const LossPlan& pl, const BothPlan& b);
hipError_t launch_both_merge(const LossArgs& a, const LossPlan& pl, const BothPlan& b);
hipError_t launch_stats_generic(const LossArgs& a, const LossPlan& pl);
hipError_t launch_grad_generic(const LossArgs& a, const LossPlan& pl);
hipError_t launch_loss_tiny(const LossArgs& a, const LossPlan& pl);      // the whole call
bool tiny_fits(int B, int P, int d);
hipError_t launch_stats_planes(const LossArgs& a, const LossPlan& pl);   // packs the inputs first
hipError_t launch_grad_planes(const LossArgs& a, const LossPlan& pl);
hipError_t launch_stats_mfma(const LossArgs& a, const LossPlan& pl);
hipError_t launch_grad_mfma(const LossArgs& a, const LossPlan& pl);
hipError_t launch_grad_online(const LossArgs& a, const LossPlan& pl);    // fused mode: dQ walk with online statistics
hipError_t launch_online_finish(const LossArgs& a, const LossPlan& pl);  // ... its splits -> lse2, row losses, dQ
hipError_t launch_loss_sum(const LossArgs& a, const LossPlan& pl);       // the fixed-order sum of the row losses alone
// symmetric loss: both directions' sums in one launch, loss = (l1 + l2) / 2, the first error word takes the second's
hipError_t launch_sym_loss_sum(const LossArgs& a1, const LossArgs& a2, const LossPlan& pl, float* loss);
hipError_t launch_stats_merge(const LossArgs& a, const LossPlan& pl);
void prof_mark_grad_kernel_done(hipStream_t s);  // measurement aid: event after the main gradient kernel(s)
bool prof_active();  // the measurement events of the loss path are being recorded
// One output of a fixed-order sum of partials (partial_reduce_kernel): up to two sources of several equal parts each.  Parts
// start at multiples of 4 floats and have room for whole vectors.
struct ReduceJob {
  void* out;
  size_t n;                 // elements
  int nsrc;
  const float* ptr[2];
  int count[2];
  size_t stride[2];         // floats between the parts of a source
  int out_bf16;             // the sum is stored as bf16 (round to nearest even)
  PosFix fix;
  int vec;                  // set by launch_reduce_jobs: `out` takes vector stores
};
// one launch for up to two outputs; loss_of / pl: it also carries the sum of the row losses of that call (see
// LossArgs::loss_with_partials)
hipError_t launch_reduce_jobs(const ReduceJob* jobs, int njobs, hipStream_t stream, const LossArgs* loss_of = nullptr,
                              const LossPlan* pl = nullptr);
// out[n] = the sum of `count` parts, `stride` floats apart
inline hipError_t launch_partial_sum(float* out, const float* part, int count, size_t stride, size_t n, hipStream_t stream) {
  ReduceJob j{};
  j.out = out; j.n = n; j.nsrc = 1; j.ptr[0] = part; j.count[0] = count; j.stride[0] = stride;
  return launch_reduce_jobs(&j, 1, stream);
}

// Workgroups are handed to the 8 XCDs round-robin by their id, and each XCD has its own L2.  This
// turns the hardware id into a task id such that each XCD works on one contiguous range of tasks
// (tasks that stream the same rows are numbered consecutively by the launchers).
__device__ __forceinline__ int xcd_task_id() {
  const int id = blockIdx.x, n = gridDim.x;
  return (n % 8 == 0) ? (id % 8) * (n / 8) + id / 8 : id;
}

// A kernel that uses more than 64 KB of dynamic LDS has to be opted in (hipFuncSetAttribute): once per kernel and
// device, remembered in `done` (a function-local array of the launcher, one per kernel instantiation).
inline hipError_t ensure_dyn_lds(const void* fn, int bytes, bool (&done)[64]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (done[dev]) return hipSuccess;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done[dev] = true;
  return e;
}

}  // namespace gc
