// What every kernel sequence of the loss / representation-gradient path shares -- the merge of split row statistics, the
// loss reduction, the fixed-order sum of split gradient partials -- and the general kernels (any d, fp32 or bf16 storage,
// fp32 FMA arithmetic) for calls whose workspace is limited (the fixed array of the entry point that allocates nothing,
// the library's buffer during a capture or on a full card, a workspace smaller than the named one): they need no packed
// inputs and no partials, and are some hundred times slower than those of loss_planes.hip (5.76 ms against 62 us at
// B = 512, P = 1024, d = 768 in fp32).
//
// Scores are kept in the base-2 domain: t_ij = s_ij * log2(e), so that
// softmax_j = 2^(t_ij - lse2_i) with lse2_i = log2 sum_j 2^t_ij (Eq. 4).
#include <type_traits>

#include "gc_common.h"

namespace gc {

template <typename T>
__device__ __forceinline__ float ldf(const T* p, size_t i);
template <>
__device__ __forceinline__ float ldf<float>(const float* p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float ldf<unsigned short>(const unsigned short* p, size_t i) { return bf2f(p[i]); }

constexpr int GT = 16;  // tile edge of the general kernels (16 x 16 scores per workgroup step)
constexpr int GK = 32;  // k-chunk staged through LDS

// One 16x16 tile of base-2 scores: thread (ty, tx) gets t for anchor row0+ty, target col0+tx.
template <typename T>
__device__ __forceinline__ float score_tile(const T* __restrict__ Q, const T* __restrict__ Pm, int B, int P, int d,
                                            int row0, int col0, float alpha2, float (*Qs)[GK + 1], float (*Ps)[GK + 1]) {
  const int tx = threadIdx.x % GT, ty = threadIdx.x / GT;
  float acc = 0.f;
  for (int k0 = 0; k0 < d; k0 += GK) {
    // 256 threads stage 16 x 32 of each operand (2 elements per thread per operand)
    for (int e = threadIdx.x; e < GT * GK; e += GT * GT) {
      int r = e / GK, k = e % GK;
      int qi = min(row0 + r, B - 1), pj = min(col0 + r, P - 1);
      bool kin = (k0 + k) < d;
      Qs[r][k] = kin ? ldf<T>(Q, (size_t)qi * d + k0 + k) : 0.f;
      Ps[r][k] = kin ? ldf<T>(Pm, (size_t)pj * d + k0 + k) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < GK; k++) acc = fmaf(Qs[ty][k], Ps[tx][k], acc);
    __syncthreads();
  }
  return acc * alpha2;
}

// Row statistics (Eq. 4's denominator, online over target tiles), one column split per blockIdx.y.
template <typename T>
__global__ void __launch_bounds__(256) stats_generic_kernel(const T* __restrict__ Q, const T* __restrict__ Pm,
                                                           const int32_t* __restrict__ pos_idx, int B, int P, int d,
                                                           float alpha2, int mask_self, int cols_per_split,
                                                           float* __restrict__ part_m, float* __restrict__ part_l,
                                                           int* __restrict__ part_idx, float* __restrict__ pos_t) {
  __shared__ float Qs[GT][GK + 1], Ps[GT][GK + 1];
  __shared__ float red_m[GT][GT], red_l[GT][GT];
  __shared__ int red_i[GT][GT];
  const int tx = threadIdx.x % GT, ty = threadIdx.x / GT;
  const int row0 = blockIdx.x * GT;
  const int split = blockIdx.y;
  const int cbeg = split * cols_per_split, cend = min(P, cbeg + cols_per_split);
  const int i = row0 + ty;
  const int ri = (i < B) ? pos_idx[i] : -1;
  float m = -INFINITY, l = 0.f;
  int best = 0x7fffffff;
  for (int col0 = cbeg; col0 < cend; col0 += GT) {
    float t = score_tile<T>(Q, Pm, B, P, d, row0, col0, alpha2, Qs, Ps);
    int j = col0 + tx;
    bool valid = (j < cend) && !(mask_self && j == i);
    // (a positive that the self-mask removes has the logit -inf: its row loss is then +inf)
    if (j < cend && j == ri && i < B) pos_t[i] = valid ? t : -INFINITY;
    if (valid) {
      if (t > m) {  // strict: ties keep the smaller index (columns are visited in increasing order)
        l = l * exp2f(m - t) + 1.f;
        m = t;
        best = j;
      } else {
        l += exp2f(t - m);
      }
    }
  }
  red_m[ty][tx] = m; red_l[ty][tx] = l; red_i[ty][tx] = best;
  __syncthreads();
  if (tx == 0 && i < B) {
    float mm = -INFINITY; int bi = 0x7fffffff;
    for (int x = 0; x < GT; x++) {
      float v = red_m[ty][x];
      if (v > mm || (v == mm && red_i[ty][x] < bi)) { mm = v; bi = red_i[ty][x]; }
    }
    float ll = 0.f;
    if (mm > -INFINITY)
      for (int x = 0; x < GT; x++) ll += red_l[ty][x] * exp2f(red_m[ty][x] - mm);
    part_m[(size_t)split * B + i] = mm;
    part_l[(size_t)split * B + i] = ll;
    part_idx[(size_t)split * B + i] = bi;
  }
}

// Merge of the split statistics of every anchor: lse2_i, row loss (Eq. 1's summand), argmax.
// LANES (a power of two >= nsplit, <= 64) consecutive lanes share one anchor, one split each, and
// combine with a fixed butterfly, so every load of the kernel is issued at once.  lse2 and the
// copy of pos_idx are padded to b_pad rows with +inf / -1, so that the gradient pass can read
// whole tiles without bounds checks (a padded row gives g = 0).
template <int LANES>
__global__ void __launch_bounds__(256) stats_merge_kernel(const float* __restrict__ part_m, const float* __restrict__ part_l,
                                                         const int* __restrict__ part_idx, float* pos_t, int pos_to_coeff,
                                                         const int32_t* __restrict__ pos_idx, int B, int P, int nsplit,
                                                         int b_pad, float* __restrict__ lse2, int32_t* __restrict__ pos_pad,
                                                         float* __restrict__ rowloss, float* __restrict__ lse_out,
                                                         int32_t* __restrict__ argmax_out, int32_t* __restrict__ inv,
                                                         int* __restrict__ shared, float* __restrict__ wexp,
                                                         int* __restrict__ wide) {
  constexpr int ROWS = 256 / LANES;
  if (shared && blockIdx.x == 0 && threadIdx.x == 0) *shared = 0;   // raised later by the gradient kernel's check
  const int s = threadIdx.x % LANES;
  const int i = blockIdx.x * ROWS + threadIdx.x / LANES;
  const bool live = (i < B) && (s < nsplit);
  float m = live ? part_m[(size_t)s * B + i] : -INFINITY;
  float l = live ? part_l[(size_t)s * B + i] : 0.f;
  int bi = live && argmax_out ? part_idx[(size_t)s * B + i] : 0x7fffffff;   // (wexp may lie where the indices would)
#pragma unroll
  for (int w = 1; w < LANES; w <<= 1) {
    const float m2 = __shfl_xor(m, w), l2 = __shfl_xor(l, w);
    const int b2 = __shfl_xor(bi, w);
    const float mn = fmaxf(m, m2);
    const float ms = (mn == -INFINITY) ? 0.f : mn;
    // both partners evaluate the same expression with the operands in the same (lower lane first) order
    const bool lower = (s & w) == 0;
    const float la = lower ? l : l2, ma = lower ? m : m2, lb = lower ? l2 : l, mb = lower ? m2 : m;
    l = la * exp2f(ma - ms) + lb * exp2f(mb - ms);
    bi = (m2 > m || (m2 == m && b2 < bi)) ? b2 : bi;
    m = mn;
  }
  if (s != 0 || i >= b_pad) return;
  if (i >= B) {
    lse2[i] = INFINITY; pos_pad[i] = -1;
    if (wexp) wexp[i] = 0.f;
    return;
  }
  const float l2 = m + log2f(l);
  lse2[i] = l2;
  if (wexp) {
    wexp[i] = exp2f(-l2 - 1.f);
    if (!(fabsf(l2) <= kWideLse)) *wide = 1;   // (zeroed by the kernel that makes the call's pairing)
  }
  const int r = pos_idx[i];
  pos_pad[i] = r;
  const bool ok = (r >= 0 && r < P);
  const float pt = ok ? pos_t[i] : 0.f;
  rowloss[i] = ok ? (l2 - pt) * kLn2 : NAN;
  if (pos_to_coeff) pos_t[i] = exp2f(pt - l2) - 1.f;   // (read by the gradient kernel of loss_planes.hip)
  if (inv && ok) inv[r] = i;   // an anchor per target; which one, when several share it, is not relied upon
  if (lse_out) lse_out[i] = l2 * kLn2;
  if (argmax_out) argmax_out[i] = bi;
}

// The same for statistics of both sides from one pass (BothPlan): sixteen rows per workgroup, sixteen threads share the slots
// of a row.  Triangle: row i has the column partials of the blocks before its own and the row partials of its block.
// Otherwise the first half of the workgroups merges the anchors' row partials, the second the targets' column partials (a
// target's positive is the anchor that inv names).
struct BothMergeArgs {
  const float* row_m; const float* row_l; const float* col_m; const float* col_l; const float* pos_t;
  const int32_t* pos; int32_t* inv;
  int triangle, n, b_pad, block, n_ablk, row_slots, cols_per_split, blocks;   // blocks: workgroups of a direction
  float* lse2[2]; float* rowloss[2]; float* wexp[2];
  int32_t* pos_pad; int* wide; int* shared;
};
__global__ void __launch_bounds__(256) both_merge_kernel(BothMergeArgs g) {
  constexpr int FLY = 8;   // loads in flight
  __shared__ float sm[4][16], sl[4][16];
  const int dir = (int)blockIdx.x >= g.blocks ? 1 : 0;
  const int row = threadIdx.x & 15, grp = threadIdx.x >> 4, w = threadIdx.x >> 6;
  const int i = ((int)blockIdx.x - dir * g.blocks) * 16 + row;
  if (blockIdx.x == 0 && threadIdx.x == 0) *g.shared = 0;
  const int blk = min(i, g.n - 1) / g.block;
  const int ncol = g.triangle ? blk : dir ? g.n_ablk : 0;
  const int nrow = g.triangle ? (g.n - g.block * blk + g.cols_per_split - 1) / g.cols_per_split : dir ? 0 : g.row_slots;
  float m = -INFINITY, l = 0.f;
  for (int s0 = grp; s0 < ncol + nrow; s0 += 16 * FLY) {
    float vm[FLY], vl[FLY];
#pragma unroll
    for (int k = 0; k < FLY; k++) {
      const int s = s0 + 16 * k;
      const bool live = i < g.n && s < ncol + nrow, col = s < ncol;
      const size_t o = live ? (size_t)(col ? s : s - ncol) * g.n + i : 0;
      vm[k] = (col ? g.col_m : g.row_m)[o]; vl[k] = (col ? g.col_l : g.row_l)[o];
      if (!live) { vm[k] = -INFINITY; vl[k] = 0.f; }
    }
    float mn = m;
#pragma unroll
    for (int k = 0; k < FLY; k++) mn = fmaxf(mn, vm[k]);
    const float ms = mn == -INFINITY ? 0.f : mn;
    l *= exp2f(m - ms);
#pragma unroll
    for (int k = 0; k < FLY; k++) l += vl[k] * exp2f(vm[k] - ms);
    m = mn;
  }
  auto merge = [&](float m2, float l2) {   // (both partners: the same value whichever is first)
    const float mn = fmaxf(m, m2), ms = mn == -INFINITY ? 0.f : mn;
    l = l * exp2f(m - ms) + l2 * exp2f(m2 - ms);
    m = mn;
  };
  merge(__shfl_xor(m, 16), __shfl_xor(l, 16));
  merge(__shfl_xor(m, 32), __shfl_xor(l, 32));
  if ((threadIdx.x & 63) < 16) { sm[w][row] = m; sl[w][row] = l; }
  __syncthreads();
  if (threadIdx.x >= 16 || i >= g.b_pad) return;
  for (int k = 1; k < 4; k++) merge(sm[k][row], sl[k][row]);
  if (i >= g.n) {
    g.lse2[dir][i] = INFINITY; g.wexp[dir][i] = 0.f;
    if (!dir) g.pos_pad[i] = -1;
    return;
  }
  int r = g.triangle ? (i ^ 1) : dir ? g.inv[i] : g.pos[i];
  if (dir && !(r >= 0 && r < g.n && g.pos[r] == i)) g.inv[i] = r = -1;   // nobody's positive: the pairing is no bijection
  if (!dir) g.pos_pad[i] = r;
  const bool ok = r >= 0 && r < g.n;
  const float pt = ok ? g.pos_t[dir ? r : i] : 0.f;
  // l's exponent to its reference: the logarithm is then of a number near 1, and its error that of one rounding of the result
  if (l > 0.f && l < INFINITY) {
    const int e = ilogbf(l);
    l = ldexpf(l, -e);
    m += (float)e;
  }
  // the sums leave the positive out: where the softmax has converged on it, the loss is log(1 + (sum of the others) / its term)
  // and not the difference of two rounded logarithms
  float l2, loss;
  const float x = l * exp2f(m - pt);
  if (ok && fabsf(pt) < INFINITY && (x <= 1.f || l == 0.f)) {
    loss = log1pf(l == 0.f ? 0.f : x);
    l2 = pt + loss * kLog2e;
  } else {
    l2 = m + log2f(ok ? l + exp2f(pt - m) : l);
    if (pt == INFINITY) l2 = NAN;   // (as any infinite score)
    loss = (l2 - pt) * kLn2;
  }
  g.lse2[dir][i] = l2;
  g.wexp[dir][i] = exp2f(-l2 - 1.f);
  if (!(fabsf(l2) <= kWideLse)) *g.wide = 1;   // (zeroed by the kernel that makes the call's pairing)
  g.rowloss[dir][i] = ok ? loss : NAN;
}
hipError_t launch_both_merge(const LossArgs& a, const LossPlan& pl, const BothPlan& b) {
  BothMergeArgs g{};
  float *rm, *rl, *cm, *cl;
  b.partials(a, pl, rm, rl, cm, cl);
  g.row_m = rm; g.row_l = rl; g.col_m = cm; g.col_l = cl;
  g.pos_t = (const float*)(a.ws + pl.off_pos); g.pos = a.pos_idx; g.inv = a.pos_inv;
  g.triangle = b.triangle; g.n = a.B; g.b_pad = pl.b_pad; g.block = b.block; g.n_ablk = b.n_ablk; g.row_slots = b.row_slots; g.cols_per_split = b.cols_per_split;
  g.blocks = (pl.b_pad + 15) / 16;
  char* const ws[2] = {a.ws, a.ws_t};
  for (int k = 0; k < (b.triangle ? 1 : 2); k++) {
    g.lse2[k] = (float*)(ws[k] + pl.off_lse2); g.rowloss[k] = (float*)(ws[k] + pl.off_rowloss); g.wexp[k] = (float*)(ws[k] + pl.off_part_idx);
  }
  g.pos_pad = (int32_t*)(a.ws + pl.off_pos_pad); g.wide = a.wide; g.shared = (int*)(a.ws + pl.off_err) + 1;
  both_merge_kernel<<<g.blocks * (b.triangle ? 1 : 2), 256, 0, a.stream>>>(g);
  // without gradients (NT-Xent with dz = NULL) no sum of partials follows that carries the row losses
  if (!a.loss_with_partials && !a.defer_loss_sum) return launch_loss_sum(a, pl);
  return hipGetLastError();
}

// loss = (1/B) sum_i rowloss_i by one workgroup; raises the error word when a row was flagged because its
// pos_idx was out of range.  The order is fixed and does not depend on the size of the workgroup: 1024 strided
// partial sums, then a binary tree over them (so the value has the same bits whichever kernel carries the sum).
struct LossSum {
  const float* rowloss;      // nullptr: nothing to do
  const int32_t* pos_idx;
  int B, P;
  float* loss;               // may be nullptr
  int* err;
};
template <int NT>  // threads of the workgroup
__device__ __forceinline__ void loss_sum_block(const LossSum& ls, float* red /* [1024] in LDS */) {
  constexpr int SL = 1024 / NT;   // partial sums per thread: slots threadIdx.x + NT * j
  float s[SL];
  int b = 0;
#pragma unroll
  for (int j = 0; j < SL; j++) s[j] = 0.f;
  // rows i0 + slot, i0 = 0, 1024, ...: the loads of four such steps are issued together, then summed in order
  for (int i0 = 0; i0 < ls.B; i0 += 4096) {
    float v[4][SL];
    int r[4][SL];
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
      for (int j = 0; j < SL; j++) {
        const int i = i0 + 1024 * k + (int)threadIdx.x + NT * j;
        const int ic = min(i, ls.B - 1);
        v[k][j] = ls.rowloss[ic];
        r[k][j] = ls.pos_idx[ic];
      }
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
      for (int j = 0; j < SL; j++) {
        const int i = i0 + 1024 * k + (int)threadIdx.x + NT * j;
        if (i < ls.B) {
          s[j] += v[k][j];
          b |= (r[k][j] < 0 || r[k][j] >= ls.P);
        }
      }
  }
#pragma unroll
  for (int j = 0; j < SL; j++) red[threadIdx.x + NT * j] = s[j];
  const int bad = __syncthreads_or(b);
  for (int w = 512; w > 0; w >>= 1) {
    for (int x = threadIdx.x; x < w; x += NT) red[x] += red[x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (ls.loss) *ls.loss = bad ? NAN : red[0] / (float)ls.B;
    *ls.err = bad ? 1 : 0;
  }
}
// symmetric loss: the second direction's sum, the mean of both, and one error word for both
template <int NT>
__device__ __forceinline__ void sym_loss_second(const LossSum& l1, const LossSum& l2, float* loss, float* red) {
  __syncthreads();                 // thread 0 has written *l1.loss and *l1.err ...
  loss_sum_block<NT>(l2, red);
  if (threadIdx.x == 0) {          // ... and reads them back itself
    if (loss) *loss = 0.5f * (*l1.loss + *l2.loss);
    if (*l2.err) *l1.err = *l2.err;
  }
}
__global__ void __launch_bounds__(1024) loss_reduce_kernel(LossSum ls) {
  __shared__ float red[1024];
  loss_sum_block<1024>(ls, red);
}

// Gradient pass, general form.  owner = the matrix whose gradient rows this workgroup owns
// (Q for Eq. 5, P for Eq. 6); the other matrix is streamed 16 rows at a time.  The owned
// 16 x d block of the output is updated in place tile by tile (one owner per row: no atomics).
template <typename T, bool OWNER_IS_Q>
__global__ void __launch_bounds__(256) grad_generic_kernel(const T* __restrict__ Q, const T* __restrict__ Pm,
                                                          const int32_t* __restrict__ pos_idx, const float* __restrict__ lse2,
                                                          int B, int P, int d, float alpha2, float out_scale, int mask_self,
                                                          float* __restrict__ out) {
  __shared__ float Qs[GT][GK + 1], Ps[GT][GK + 1];
  __shared__ float g[GT][GT + 1];  // g[owner row][stream row]
  const int tx = threadIdx.x % GT, ty = threadIdx.x / GT;
  const int own0 = blockIdx.x * GT;
  const int n_own = OWNER_IS_Q ? B : P, n_str = OWNER_IS_Q ? P : B;
  const T* S = OWNER_IS_Q ? Pm : Q;
  bool first = true;
  for (int str0 = 0; str0 < n_str; str0 += GT) {
    const int row0 = OWNER_IS_Q ? own0 : str0;  // anchors on ty
    const int col0 = OWNER_IS_Q ? str0 : own0;  // targets on tx
    float t = score_tile<T>(Q, Pm, B, P, d, row0, col0, alpha2, Qs, Ps);
    int i = row0 + ty, j = col0 + tx;
    float gv = 0.f;
    if (i < B && j < P && !(mask_self && i == j)) {
      gv = exp2f(t - lse2[i]) - ((pos_idx[i] == j) ? 1.f : 0.f);
    }
    if (OWNER_IS_Q) g[ty][tx] = gv * out_scale; else g[tx][ty] = gv * out_scale;
    __syncthreads();
    for (int e = threadIdx.x; e < GT * d; e += 256) {
      int r = e / d, c = e % d;
      if (own0 + r < n_own) {
        float acc = 0.f;
        for (int b = 0; b < GT; b++) {
          int sr = min(str0 + b, n_str - 1);  // g is 0 past the end
          acc = fmaf(g[r][b], ldf<T>(S, (size_t)sr * d + c), acc);
        }
        size_t o = (size_t)(own0 + r) * d + c;
        out[o] = first ? acc : out[o] + acc;
      }
    }
    first = false;
    __syncthreads();
  }
}

// Fixed-order sums of split partials: out[e] = sum over sources s, over parts k < count[s] of ptr[s][k * stride[s] + e],
// up to two outputs (dq and dp) in one launch.  With a loss sum attached the grid has one more workgroup, the first (so
// that it runs beside the others), which carries it (it has nothing to do with the partial sums; it only saves a launch
// on the path that needs both).
struct ReduceArgs {
  ReduceJob job[2]; unsigned blocks0; LossSum ls;
  LossSum ls2; float* sym_loss;   // with ls: the other direction of the symmetric loss, and the mean's place
};
// coefficient of the positive of anchor i (target r), see PosFix
__device__ __forceinline__ float pos_coeff(const PosFix& f, int i, int r) {
  const float t = f.pos_t[i];
  float c = exp2f(t - f.lse2[i]);
  if (f.lse2_t) c = 0.5f * (c + exp2f(t - f.lse2_t[r]));
  return f.scale * (c - 1.f);
}
__device__ __forceinline__ void add_row4(f32x4& acc, float c, const unsigned short* row, int col) {
  const s16x4 v = *(const s16x4*)(row + col);
#pragma unroll
  for (int k = 0; k < 4; k++) acc[k] += c * bf2f((unsigned short)v[k]);
}
// What a workgroup of the sum kernel keeps of up to 1024 anchors that share a target: the anchor, its target and coefficient
constexpr int kListLen = 1024, kListPer = kListLen / 256;
struct SharedList { int anchor[kListLen]; int row[kListLen]; float c[kListLen]; int cnt[kListPer][4]; };
// Some target is the positive of several anchors: every anchor that names one of the rows of this workgroup's elements
// (first .. last), in index order.  The workgroup looks through the anchors together, 1024 at a time (four a thread, loaded
// together: at 256 a time each round's loads and barriers are a latency of their own, 14.3 us for the sums of 1021 x 4099 x 384,
// now 11.9), and keeps the matches with their coefficients (in index order: ballot and prefix inside a wave, waves one after the
// other) in LDS; each thread then adds those of its own rows, eight loads in flight.  (A scan by every thread for itself took
// 179 us there, and 1.0 ms where 2700 anchors share one target of 300.)  Workgroups none of whose rows is named, the most of
// them, are done at once.
__device__ __forceinline__ void add_shared_positives(f32x4& acc, const PosFix& fx, size_t first, size_t last, int row, int col, bool live,
                                                     SharedList& list) {
  const int row0 = (int)(first / (size_t)fx.d), row1 = (int)(last / (size_t)fx.d);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int r[kListPer];
  auto load = [&](int i0) {
#pragma unroll
    for (int k = 0; k < kListPer; k++) {
      const int i = i0 + 256 * k + (int)threadIdx.x;
      r[k] = i < fx.B ? fx.pos[i] : -1;
    }
  };
  load(0);   // (in flight while the check below waits for its own loads)
  bool named = false;
  if (live) {   // the merge records one of the anchors of every named target (whatever the workspace held, if none: checked)
    const int i = fx.inv[row];
    named = i >= 0 && i < fx.B && fx.pos[i] == row;
  }
  if (!__syncthreads_or(named)) return;
  for (int i0 = 0; i0 < fx.B; i0 += kListLen) {
    if (i0) load(i0);
    unsigned long long mask[kListPer];
#pragma unroll
    for (int k = 0; k < kListPer; k++) {
      mask[k] = __builtin_amdgcn_ballot_w64(r[k] >= row0 && r[k] <= row1);
      if (lane == 0) list.cnt[k][w] = __builtin_popcountll(mask[k]);
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int k = 0; k < kListPer; k++) {
      int base = total;
#pragma unroll
      for (int x = 0; x < 4; x++) {
        const int n = list.cnt[k][x];
        base += x < w ? n : 0;
        total += n;
      }
      if (r[k] >= row0 && r[k] <= row1) {
        const int at = base + __builtin_popcountll(mask[k] & ((1ull << lane) - 1ull)), i = i0 + 256 * k + (int)threadIdx.x;
        list.anchor[at] = i; list.row[at] = r[k]; list.c[at] = pos_coeff(fx, i, r[k]);
      }
    }
    __syncthreads();
    constexpr int FLY = 8;
    for (int k0 = 0; k0 < total; k0 += FLY) {
      s16x4 o[FLY];   // (loaded whether or not the anchor is this row's: a load behind a condition is waited for one by one)
      bool mine[FLY];
      float c[FLY];
#pragma unroll
      for (int k = 0; k < FLY; k++) {
        const int at = min(k0 + k, total - 1);
        mine[k] = k0 + k < total && live && list.row[at] == row;
        c[k] = list.c[at];
        o[k] = *(const s16x4*)(fx.other + (size_t)list.anchor[at] * fx.d + col);
      }
#pragma unroll
      for (int k = 0; k < FLY; k++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const float sum = acc[e] + c[k] * bf2f((unsigned short)o[k][e]);
          acc[e] = mine[k] ? sum : acc[e];
        }
    }
    __syncthreads();   // the list and the counts are free again
  }
}
// Four elements per thread.  Bound by memory: 88 MB in 16 us for the dP sums of 4096 x 8192 x 768, most of it out of the
// memory-side cache, with eight waves per SIMD (18.5 us with six or with 8 elements per thread).
// Partials are loaded past the caches, results stored through them.  With inputs that change from call to call the loads
// matter, 241.1 us against 247.3 at 4096 x 8192 x 768 (324 and 337 for the bilinear loss); results stored past the caches as
// well gain nothing there (241.4) and 1 % at 1021 x 4099 x 384 (63.8 and 64.4), but whoever reads dq and dp next pays for it:
// with a cast of both behind the call 258.6 and 256.8 us, 72.1 and 71.5.
// (JOBS = 1: every argument sits at a known place, so they are all loaded at once; picking one of two costs 2 us here.)
template <int JOBS>
__global__ void __launch_bounds__(256, 8) partial_reduce_kernel(ReduceArgs a) {
  __shared__ union { float red[1024]; SharedList list; } lds;
  unsigned block = blockIdx.x;
  if (a.ls.rowloss) {
    if (block == 0) {
      loss_sum_block<256>(a.ls, lds.red);
      if (JOBS > 1 && a.ls2.rowloss) sym_loss_second<256>(a.ls, a.ls2, a.sym_loss, lds.red);
      return;
    }
    block--;
  }
  const bool second = JOBS > 1 && block >= a.blocks0;
  if (second) block -= a.blocks0;
  const ReduceJob& j = second ? a.job[1] : a.job[0];
  const PosFix& fx = j.fix;
  const size_t n4 = (j.n + 3) / 4, e0 = (size_t)block * 256, e = e0 + threadIdx.x;
  const bool live = e < n4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (live) {   // (partials have room for whole vectors)
    int k = 0;
    for (; k + 4 <= j.count[0]; k += 4) {   // four loads in flight, added in order
      f32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; i++) v[i] = __builtin_nontemporal_load((const f32x4*)(j.ptr[0] + (size_t)(k + i) * j.stride[0]) + e);
#pragma unroll
      for (int i = 0; i < 4; i++) acc += v[i];
    }
    for (; k < j.count[0]; k++) acc += __builtin_nontemporal_load((const f32x4*)(j.ptr[0] + (size_t)k * j.stride[0]) + e);
    if (j.nsrc > 1)
      for (int k = 0; k < j.count[1]; k++) acc += ((const f32x4*)(j.ptr[1] + (size_t)k * j.stride[1]))[e];
  }
  if (fx.mode) {   // the positive's term, in fp32, after the partials (d is a multiple of 4 here)
    const size_t first = e0 * 4;
    int row, col;
    if (j.n <= 0xffffffffu) {   // one 32-bit division
      const unsigned x = (unsigned)(e * 4), r = x / (unsigned)fx.d;
      row = (int)r; col = (int)(x - r * (unsigned)fx.d);
    } else {
      row = (int)(e * 4 / (size_t)fx.d); col = (int)(e * 4 % (size_t)fx.d);
    }
    if (fx.mode == 1) {
      const int r = live ? fx.pos[row] : -1;
      if (r >= 0 && r < fx.P) add_row4(acc, pos_coeff(fx, row, r), fx.other + (size_t)r * fx.d, col);
    } else if (*fx.shared == 0) {
      const int i = live ? fx.inv[row] : -1;   // whatever the workspace held if no anchor names this target: checked
      if (i >= 0 && i < fx.B && fx.pos[i] == row) add_row4(acc, pos_coeff(fx, i, row), fx.other + (size_t)i * fx.d, col);
    } else {
      add_shared_positives(acc, fx, first, (e0 + 256 < n4 ? e0 + 256 : n4) * 4 - 1, row, col, live, lds.list);
    }
  }
  if (!live) return;
  if (4 * e + 4 <= j.n && j.vec) {
    if (j.out_bf16) {
      typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
      ((bf16x4_t*)j.out)[e] = __builtin_convertvector(acc, bf16x4_t);
    } else {
      ((f32x4*)j.out)[e] = acc;
    }
  } else {   // the last elements of an odd count, or an output that is only aligned to its elements
    for (int k = 0; k < 4 && 4 * e + k < j.n; k++) {
      if (j.out_bf16) ((__bf16*)j.out)[4 * e + k] = (__bf16)acc[k];
      else ((float*)j.out)[4 * e + k] = acc[k];
    }
  }
}

// Fused mode: merge of what the splits of the online dQ walk left per anchor (reference, sum 2^(t - reference), and
// when the arg-max is asked for the true maximum with its first index) into lse2_i, the row loss and the arg-max, and
//   dQ_i = sum_s 2^(ref_s,i - lse2_i) part_s,i + (alpha / B) (p_{i r_i} - 1) p_{r_i}
// where part_s,i = (alpha / B) sum_{j in split s, j != r_i} 2^(t_ij - ref_s,i) p_j (Eq. 5; the positive's own term is
// formed here in fp32, so a softmax that has converged on the positive does not cancel in bf16).  Splits are
// combined in index order.  64 threads per anchor, 4 anchors per workgroup.
struct FinishArgs {
  const float* on_ref; const float* on_l; const float* on_best; const int* on_idx; const float* on_pos;
  const int32_t* pos_idx; const unsigned short* P;
  const float* part; size_t part_stride;
  int nsq, B, Pn, d, b_pad;
  float out_scale;
  float* lse2; int32_t* pos_pad; float* rowloss; float* lse_out; int32_t* argmax_out; float* dq;
  int dq_bf16;   // dq points to bf16 elements
  int32_t* inv; int* shared;   // an anchor per target and the "several anchors share a target" word (see PosFix)
};
__global__ void __launch_bounds__(256) online_finish_kernel(FinishArgs f) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (blockIdx.x == 0 && threadIdx.x == 0) *f.shared = 0;   // raised later by the dP walk's check
  if (i >= f.b_pad) return;
  if (i >= f.B) {
    if (lane == 0) { f.lse2[i] = INFINITY; f.pos_pad[i] = -1; }
    return;
  }
  // every load of the row's statistics is issued before the first result is needed
  float sl[16], sr[16];
#pragma unroll
  for (int s = 0; s < 16; s++) {
    const bool live = s < f.nsq;
    const size_t o = (size_t)(live ? s : 0) * f.B + i;
    sl[s] = live ? f.on_l[o] : 0.f; sr[s] = live ? f.on_ref[o] : -INFINITY;
  }
  const int r = f.pos_idx[i];
  const bool ok = (r >= 0 && r < f.Pn);
  const int r_safe = ok ? r : 0;
  const float pos = f.on_pos[i];
  float M = -INFINITY;
#pragma unroll
  for (int s = 0; s < 16; s++) M = fmaxf(M, sr[s]);
  float L = 0.f;
  if (M > -INFINITY) {
#pragma unroll
    for (int s = 0; s < 16; s++) L += sl[s] * exp2f(sr[s] - M);   // dead splits: 0 * 2^-inf = 0
  }
  const float l2 = M + log2f(L);
  if (lane == 0) {
    f.lse2[i] = l2;
    f.pos_pad[i] = r;
    f.rowloss[i] = ok ? (l2 - pos) * kLn2 : NAN;
    if (ok) f.inv[r] = i;
    if (f.lse_out) f.lse_out[i] = l2 * kLn2;
    if (f.argmax_out) {
      float bv = -INFINITY; int bi = 0x7fffffff;
      for (int s = 0; s < f.nsq; s++) {
        const float v = f.on_best[(size_t)s * f.B + i];
        const int idx = f.on_idx[(size_t)s * f.B + i];
        if (v > bv || (v == bv && idx < bi)) { bv = v; bi = idx; }
      }
      f.argmax_out[i] = bi;
    }
  }
  if (!f.dq) return;
  float w[16];
#pragma unroll
  for (int s = 0; s < 16; s++) w[s] = exp2f(sr[s] - l2);
  // coefficient of the positive: p_{i r_i} - 1
  const float cpos = ok ? f.out_scale * (exp2f(pos - l2) - 1.f) : 0.f;
  for (int c = lane; c < f.d / 4; c += 64) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 16; s++)
      if (s < f.nsq) acc += w[s] * __builtin_nontemporal_load((const f32x4*)(f.part + (size_t)s * f.part_stride + (size_t)i * f.d) + c);
    const s16x4 pv = ((const s16x4*)(f.P + (size_t)r_safe * f.d))[c];
#pragma unroll
    for (int e = 0; e < 4; e++) acc[e] += cpos * bf2f((unsigned short)pv[e]);
    if (f.dq_bf16) {
      typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
      ((bf16x4_t*)((__bf16*)f.dq + (size_t)i * f.d))[c] = __builtin_convertvector(acc, bf16x4_t);
    } else {
      ((f32x4*)(f.dq + (size_t)i * f.d))[c] = acc;
    }
  }
}

hipError_t launch_online_finish(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  FinishArgs f{};
  f.on_ref = (const float*)(ws + pl.off_on_ref); f.on_best = (const float*)(ws + pl.off_part_m);
  f.on_l = (const float*)(ws + pl.off_part_l); f.on_idx = (const int*)(ws + pl.off_part_idx);
  f.on_pos = (const float*)(ws + pl.off_pos); f.pos_idx = a.pos_idx; f.P = (const unsigned short*)a.p;
  f.part = (const float*)(ws + pl.off_dq_part); f.part_stride = (size_t)a.B * a.d;
  f.nsq = pl.fz_nsq; f.B = a.B; f.Pn = a.P; f.d = a.d; f.b_pad = pl.b_pad;
  f.out_scale = a.alpha / (float)a.B * (a.grad_mul != 0.f ? a.grad_mul : 1.f);
  f.lse2 = (float*)(ws + pl.off_lse2); f.pos_pad = (int32_t*)(ws + pl.off_pos_pad); f.rowloss = (float*)(ws + pl.off_rowloss);
  f.lse_out = a.lse; f.argmax_out = a.argmax; f.dq = a.dq; f.dq_bf16 = (a.flags & GC_CACHE_BF16) ? 1 : 0;
  f.inv = (int32_t*)(ws + pl.off_inv); f.shared = (int*)(ws + pl.off_err) + 1;
  online_finish_kernel<<<(pl.b_pad + 3) / 4, 256, 0, a.stream>>>(f);
  return hipGetLastError();
}

static LossSum loss_sum_of(const LossArgs& a, const LossPlan& pl) {
  LossSum ls{};
  ls.rowloss = (const float*)(a.ws + pl.off_rowloss); ls.pos_idx = a.pos_idx; ls.B = a.B; ls.P = a.P;
  ls.loss = a.loss; ls.err = (int*)(a.ws + pl.off_err);
  return ls;
}

hipError_t launch_reduce_jobs(const ReduceJob* jobs, int njobs, hipStream_t stream, const LossArgs* loss_of, const LossPlan* pl) {
  ReduceArgs a{};
  unsigned blocks[2] = {0, 0};
  for (int k = 0; k < njobs; k++) {
    a.job[k] = jobs[k];
    a.job[k].vec = ((uintptr_t)jobs[k].out & (jobs[k].out_bf16 ? 7 : 15)) == 0;
    if (jobs[k].fix.mode && (jobs[k].n % 4 || jobs[k].fix.d % 4)) return hipErrorInvalidValue;   // rows of whole vectors only
    blocks[k] = (unsigned)(((jobs[k].n + 3) / 4 + 255) / 256);
  }
  if (loss_of && loss_of->sym[0]) {   // (two jobs: both gradients of the symmetric loss)
    a.ls = loss_sum_of(*loss_of->sym[0], *pl);
    a.ls2 = loss_sum_of(*loss_of->sym[1], *pl);
    a.sym_loss = loss_of->sym_loss;
  } else if (loss_of) {
    a.ls = loss_sum_of(*loss_of, *pl);
  }
  a.blocks0 = blocks[0];
  const unsigned n = blocks[0] + blocks[1] + (loss_of ? 1 : 0);
  if (n && njobs > 1) partial_reduce_kernel<2><<<dim3(n), 256, 0, stream>>>(a);
  else if (n) partial_reduce_kernel<1><<<dim3(n), 256, 0, stream>>>(a);
  return hipGetLastError();
}

template <typename T>
static hipError_t stats_generic_t(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  dim3 grid((a.B + GT - 1) / GT, pl.stat_splits);
  stats_generic_kernel<T><<<grid, 256, 0, a.stream>>>((const T*)a.q, (const T*)a.p, a.pos_idx, a.B, a.P, a.d,
                                                      a.alpha * kLog2e, (a.flags & GC_MASK_SELF) ? 1 : 0,
                                                      pl.stat_cols_per_split, (float*)(ws + pl.off_part_m),
                                                      (float*)(ws + pl.off_part_l), (int*)(ws + pl.off_part_idx),
                                                      (float*)(ws + pl.off_pos));
  return hipGetLastError();
}
hipError_t launch_stats_generic(const LossArgs& a, const LossPlan& pl) {
  return a.dt == GC_F32 ? stats_generic_t<float>(a, pl) : stats_generic_t<unsigned short>(a, pl);
}

hipError_t launch_loss_sum(const LossArgs& a, const LossPlan& pl) {
  loss_reduce_kernel<<<1, 1024, 0, a.stream>>>(loss_sum_of(a, pl));
  return hipGetLastError();
}

__global__ void __launch_bounds__(1024) sym_loss_reduce_kernel(LossSum l1, LossSum l2, float* loss) {
  __shared__ float red[1024];
  loss_sum_block<1024>(l1, red);
  sym_loss_second<1024>(l1, l2, loss, red);
}
hipError_t launch_sym_loss_sum(const LossArgs& a1, const LossArgs& a2, const LossPlan& pl, float* loss) {
  sym_loss_reduce_kernel<<<1, 1024, 0, a1.stream>>>(loss_sum_of(a1, pl), loss_sum_of(a2, pl), loss);
  return hipGetLastError();
}

hipError_t launch_stats_merge(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  auto merge = [&](auto lanes_tag) {
    constexpr int LANES = decltype(lanes_tag)::value;
    constexpr int ROWS = 256 / LANES;
    stats_merge_kernel<LANES><<<(pl.b_pad + ROWS - 1) / ROWS, 256, 0, a.stream>>>(
        (const float*)(ws + pl.off_part_m), (const float*)(ws + pl.off_part_l), (const int*)(ws + pl.off_part_idx),
        (float*)(ws + pl.off_pos), pl.route == ROUTE_PLANES ? 1 : 0, a.pos_idx, a.B, a.P, pl.stat_splits, pl.b_pad, (float*)(ws + pl.off_lse2),
        (int32_t*)(ws + pl.off_pos_pad), (float*)(ws + pl.off_rowloss), a.lse, a.argmax,
        pl.use_mfma ? (int32_t*)(ws + pl.off_inv) : nullptr, pl.use_mfma ? (int*)(ws + pl.off_err) + 1 : nullptr,
        a.wexp, a.wide);
  };
  if (pl.stat_splits <= 1) merge(std::integral_constant<int, 1>{});
  else if (pl.stat_splits <= 4) merge(std::integral_constant<int, 4>{});
  else if (pl.stat_splits <= 16) merge(std::integral_constant<int, 16>{});
  else merge(std::integral_constant<int, 64>{});
  // the sum of the row losses: by a launch of its own, unless a sum of gradient partials follows that carries it
  if (!a.loss_with_partials && !a.defer_loss_sum) loss_reduce_kernel<<<1, 1024, 0, a.stream>>>(loss_sum_of(a, pl));
  return hipGetLastError();
}

template <typename T>
static hipError_t grad_generic_t(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  const float* lse2 = (const float*)(ws + pl.off_lse2);
  const float alpha2 = a.alpha * kLog2e, osc = a.alpha / (float)a.B * (a.grad_mul != 0.f ? a.grad_mul : 1.f);
  const int ms = (a.flags & GC_MASK_SELF) ? 1 : 0;
  float* dq = a.dz ? (float*)(ws + pl.off_dq_part) : a.dq;
  float* dp = a.dz ? (float*)(ws + pl.off_dp_part) : a.dp;
  if (dq)
    grad_generic_kernel<T, true><<<(a.B + GT - 1) / GT, 256, 0, a.stream>>>((const T*)a.q, (const T*)a.p, a.pos_idx, lse2,
                                                                           a.B, a.P, a.d, alpha2, osc, ms, dq);
  if (dp)
    grad_generic_kernel<T, false><<<(a.P + GT - 1) / GT, 256, 0, a.stream>>>((const T*)a.q, (const T*)a.p, a.pos_idx, lse2,
                                                                            a.B, a.P, a.d, alpha2, osc, ms, dp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  prof_mark_grad_kernel_done(a.stream);
  if (a.dz) {
    ReduceJob j{};
    j.out = a.dz; j.n = (size_t)a.B * a.d; j.nsrc = 2;
    j.ptr[0] = dq; j.ptr[1] = dp; j.count[0] = j.count[1] = 1;
    return launch_reduce_jobs(&j, 1, a.stream);
  }
  return hipSuccess;
}
hipError_t launch_grad_generic(const LossArgs& a, const LossPlan& pl) {
  return a.dt == GC_F32 ? grad_generic_t<float>(a, pl) : grad_generic_t<unsigned short>(a, pl);
}


// ---- a handful of scores -------------------------------------------------------------------------------------------------
// The whole call in one workgroup: both inputs, the scores and then the coefficients stay in LDS.  Such a call is bound by
// its launches (8 x 16 x 64 took five, 18 us of kernels); one workgroup is faster than the kernels of loss_planes.hip up
// to some 2^17 products: 12.2 us at 8 x 16 x 64, 12.9 at 32 x 32 x 64 and 19 at 32 x 64 x 64 against 26; 32 at 8 x 32 x 768
// against 55, but 34 at 64 x 64 x 64 against 26.
constexpr long long kTinyWork = 1ll << 17;   // at small widths, see tiny_fits
struct TinyArgs {
  const void* q; const void* p; const int32_t* pos_idx;
  int B, P, d, ld;                      // ld: odd row stride of the inputs in LDS
  float alpha2, out_scale;
  int mask_self;
  float* loss; float* dq; float* dp; float* dz; float* lse; int32_t* argmax; float* rowloss; int* err;
};
template <typename T>
__global__ void __launch_bounds__(1024) loss_tiny_kernel(TinyArgs g) {
  extern __shared__ __attribute__((aligned(16))) float tiny_lds[];
  float* Q = tiny_lds;
  float* Pm = Q + g.B * g.ld;
  float* S = Pm + g.P * g.ld;           // [B][P + 1]
  float* rl = S + g.B * (g.P + 1);      // [B] row losses
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ls = g.P + 1;
  for (int e = tid; e < g.B * g.d; e += 1024) Q[(e / g.d) * g.ld + e % g.d] = ldf<T>((const T*)g.q, e);
  for (int e = tid; e < g.P * g.d; e += 1024) Pm[(e / g.d) * g.ld + e % g.d] = ldf<T>((const T*)g.p, e);
  int bad = 0;
  for (int i = tid; i < g.B; i += 1024) bad |= g.pos_idx[i] < 0 || g.pos_idx[i] >= g.P;
  bad = __syncthreads_or(bad);
  for (int e = tid; e < g.B * g.P; e += 1024) {
    const int i = e / g.P, j = e % g.P;
    const float* a = Q + i * g.ld;
    const float* b = Pm + j * g.ld;
    float s = 0.f;
#pragma unroll 8
    for (int k = 0; k < g.d; k++) s = fmaf(a[k], b[k], s);
    S[i * ls + j] = (g.mask_self && i == j) ? -INFINITY : s * g.alpha2;
  }
  __syncthreads();
  for (int i = wave; i < g.B; i += 16) {   // a wave per anchor
    float* row = S + i * ls;
    float m = -INFINITY;
    int best = 0x7fffffff;
    for (int j = lane; j < g.P; j += 64)
      if (row[j] > m) { m = row[j]; best = j; }   // strict: the smallest index of this lane
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) {
      const float m2 = __shfl_xor(m, w);
      const int b2 = __shfl_xor(best, w);
      if (m2 > m || (m2 == m && b2 < best)) { m = m2; best = b2; }
    }
    const float ms = (m == -INFINITY) ? 0.f : m;
    float l = 0.f;
    for (int j = lane; j < g.P; j += 64) l += exp2f(row[j] - ms);
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) l += __shfl_xor(l, w);
    const float lse2 = ms + log2f(l);
    const int r = g.pos_idx[i];
    const bool ok = r >= 0 && r < g.P;
    if (lane == 0) {
      rl[i] = ok ? (lse2 - row[ok ? r : 0]) * kLn2 : NAN;
      g.rowloss[i] = rl[i];
      if (g.lse) g.lse[i] = lse2 * kLn2;
      if (g.argmax) g.argmax[i] = best;
    }
    for (int j = lane; j < g.P; j += 64)
      row[j] = (g.mask_self && i == j) ? 0.f : exp2f(row[j] - lse2) - (j == r ? 1.f : 0.f);
  }
  __syncthreads();
  if (wave == 0) {   // mean of the row losses, in a fixed order
    float s = 0.f;
    for (int i = lane; i < g.B; i += 64) s += rl[i];
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) s += __shfl_xor(s, w);
    if (lane == 0) {
      if (g.loss) *g.loss = bad ? NAN : s / (float)g.B;
      *g.err = bad ? 1 : 0;
    }
  }
  if (g.dq || g.dz)
    for (int e = tid; e < g.B * g.d; e += 1024) {
      const int i = e / g.d, c = e % g.d;
      float s = 0.f;
#pragma unroll 8
      for (int j = 0; j < g.P; j++) s = fmaf(S[i * ls + j], Pm[j * g.ld + c], s);
      if (g.dz) {   // (B == P, one input) + the target's part of the same row
        float t = 0.f;
#pragma unroll 8
        for (int j = 0; j < g.B; j++) t = fmaf(S[j * ls + i], Q[j * g.ld + c], t);
        g.dz[e] = s * g.out_scale + t * g.out_scale;
      } else {
        g.dq[e] = s * g.out_scale;
      }
    }
  if (g.dp)
    for (int e = tid; e < g.P * g.d; e += 1024) {
      const int j = e / g.d, c = e % g.d;
      float s = 0.f;
#pragma unroll 8
      for (int i = 0; i < g.B; i++) s = fmaf(S[i * ls + j], Q[i * g.ld + c], s);
      g.dp[e] = s * g.out_scale;
    }
}
static size_t tiny_lds_bytes(int B, int P, int d) { return ((size_t)(B + P) * (d | 1) + (size_t)B * (P + 1) + B) * 4; }
bool tiny_fits(int B, int P, int d) {
  if (B > 1024 || P > 1024 || d > 4096) return false;
  // (the other kernels walk the width in one chain: 26 us at d = 64, 55 at 768)
  return (long long)B * P * d <= kTinyWork + kTinyWork * d / 384 && tiny_lds_bytes(B, P, d) <= 150 * 1024;
}
template <typename T>
static hipError_t tiny_t(const TinyArgs& g, size_t lds, hipStream_t s) {
  static bool done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)loss_tiny_kernel<T>, 150 * 1024, done); e != hipSuccess) return e;
  loss_tiny_kernel<T><<<1, 1024, lds, s>>>(g);
  return hipGetLastError();
}
hipError_t launch_loss_tiny(const LossArgs& a, const LossPlan& pl) {
  TinyArgs g{};
  g.q = a.q; g.p = a.p; g.pos_idx = a.pos_idx; g.B = a.B; g.P = a.P; g.d = a.d; g.ld = a.d | 1;
  g.alpha2 = a.alpha * kLog2e; g.out_scale = a.alpha / (float)a.B * (a.grad_mul != 0.f ? a.grad_mul : 1.f);
  g.mask_self = (a.flags & GC_MASK_SELF) ? 1 : 0;
  g.loss = a.defer_loss_sum ? nullptr : a.loss; g.dq = a.dq; g.dp = a.dp; g.dz = a.dz; g.lse = a.lse; g.argmax = a.argmax;
  g.rowloss = (float*)(a.ws + pl.off_rowloss); g.err = (int*)(a.ws + pl.off_err);
  const size_t lds = tiny_lds_bytes(a.B, a.P, a.d);
  return a.dt == GC_F32 ? tiny_t<float>(g, lds, a.stream) : tiny_t<unsigned short>(g, lds, a.stream);
}

}  // namespace gc
