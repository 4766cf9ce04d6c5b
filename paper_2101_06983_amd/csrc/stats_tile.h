// Row statistics of 32 x 32 score tiles whose contraction was split over the four waves of a workgroup: what the kernels
// for few scores (bf16 widths and planes) share.
#pragma once
#include "gc_common.h"

namespace gc {

__device__ __forceinline__ void stat_merge(float& m, float& l, int& idx, float m2, float l2, int idx2) {
  // (m, idx): larger value wins, ties to the smaller index
  bool take = (m2 > m) || (m2 == m && idx2 < idx);
  float mn = fmaxf(m, m2);
  float ms = (mn == -INFINITY) ? 0.f : mn;
  l = l * fast_exp2(m - ms) + l2 * fast_exp2(m2 - ms);
  idx = take ? idx2 : idx;
  m = mn;
}

struct StatsSmallArgs {
  const unsigned short* Q; const unsigned short* P; const int32_t* pos_idx;
  int B, Pn, d, n_ablk, tiles, tiles_per_split, mask_self;
  float alpha2;
  float* part_m; float* part_l; int* part_idx; float* pos_t;
  int32_t* inv; int* shared;   // where no merge follows: an anchor per target, and the word that the gradient kernel may raise
};
struct StatTileLds {
  float red[4][kStatTile][kStatTile + 1];                          // partial tiles of the four waves: [target][anchor]
  float m[256 / kStatTile][kStatTile], l[256 / kStatTile][kStatTile];   // per part of the targets: maximum, sum, index
  int idx[256 / kStatTile][kStatTile];
};
// Thread (part, n) of 256 takes targets TP part .. of anchor n.  EXACT: terms by the library's exp2f, which keeps results
// below 2^-126 that the hardware's flushes.  (The parts are merged by the hardware's either way: such a weight is nothing
// beside the 1 or more of the part with the maximum, and exp2f there costs 0.4 us of the 50 of 512 x 1024 x 1024.)
template <bool EXACT>
struct StatTile {
  static constexpr int T = kStatTile, PARTS = 256 / T, TP = T / PARTS;
  float m = -INFINITY, l = 0.f;
  int best = 0x7fffffff, en, part, a, r;
  static __device__ __forceinline__ float ex(float x) { return EXACT ? exp2f(x) : fast_exp2(x); }
  __device__ __forceinline__ StatTile(const StatsSmallArgs& g, int a0) {
    en = threadIdx.x % T; part = threadIdx.x / T; a = a0 + en;
    r = a < g.B ? g.pos_idx[a] : -1;
  }
  // this wave's partial products of the tile of targets j0 .. (targets on M: lane ln holds anchor ln)
  static __device__ __forceinline__ void put(StatTileLds& s, int wave, const f32x16& acc) {
    const int lane = threadIdx.x & 63, h = lane >> 5, ln = lane & 31;
#pragma unroll
    for (int e = 0; e < 16; e++) s.red[wave][8 * (e >> 2) + 4 * h + (e & 3)][ln] = acc[e];
  }
  // after a barrier; the caller puts another one behind it
  __device__ __forceinline__ void tile(const StatsSmallArgs& g, const StatTileLds& s, int j0) {
    float v[TP], mt = -INFINITY;
    int bt = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < TP; e++) {
      const int row = part * TP + e, j = j0 + row;
      float x = (((s.red[0][row][en] + s.red[1][row][en]) + s.red[2][row][en]) + s.red[3][row][en]) * g.alpha2;
      if (j >= g.Pn || (g.mask_self && j == a)) x = -INFINITY;
      // (a positive that the self-mask removes has the logit -inf: its row loss is then +inf)
      if (j == r && j < g.Pn && a < g.B) g.pos_t[a] = x;
      v[e] = x;
      if (x > mt) { mt = x; bt = j; }   // strict: the smallest index attaining the maximum
    }
    const float mn = fmaxf(m, mt), ms = (mn == -INFINITY) ? 0.f : mn;
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < TP; e++) sum += ex(v[e] - ms);
    l = l * ex(m - ms) + sum;
    if (mt > m) best = bt;
    m = mn;
  }
  __device__ __forceinline__ void finish(const StatsSmallArgs& g, StatTileLds& s, int split) {
    s.m[part][en] = m; s.l[part][en] = l; s.idx[part][en] = best;
    __syncthreads();
    if (threadIdx.x < T && a < g.B) {   // part 0 of every anchor: the others in order
#pragma unroll
      for (int k = 1; k < PARTS; k++) stat_merge(m, l, best, s.m[k][en], s.l[k][en], s.idx[k][en]);
      const size_t o = (size_t)split * g.B + a;
      g.part_m[o] = m; g.part_l[o] = l; g.part_idx[o] = best;
    }
  }
};
// The gradient kernels for few scores merge the split statistics of the rows they need (merges_itself): one launch of 3.5 us
// and its gap less.  The workgroups that own a block of anchors with `write` leave what the merge kernel would.
struct FewMerge {
  int splits;                 // 0: already merged
  const float* part_m; const float* part_l; const int* part_idx; const float* pos_t;
  float* lse2; float* rowloss; float* lse_out; int32_t* argmax_out;
};
// Anchors first .. first + n - 1 (n <= kFewMergeRows) by a workgroup of TH: TH / n2 threads a row (n2: n rounded up to a power
// of two from 32), eight splits' loads in flight each.  The constructor issues the first loads; what the caller loads between
// it and finish() is in flight beside them.
template <bool EXACT, int TH = 256>
struct StatMerge {
  static constexpr int FLY = 8;
  static __device__ __forceinline__ float ex(float v) { return EXACT ? exp2f(v) : fast_exp2(v); }
  int lg, grps, row, grp, i, r;
  bool live, write;
  float pt, vm[FLY], vl[FLY];
  int vi[FLY];
  __device__ __forceinline__ void load(const FewMerge& fm, int B, int s0) {
    const bool want_idx = write && fm.argmax_out;
#pragma unroll
    for (int k = 0; k < FLY; k++) {
      const bool in = s0 + k < fm.splits;
      const size_t o = (size_t)(in ? s0 + k : 0) * B + i;
      vm[k] = fm.part_m[o]; vl[k] = fm.part_l[o]; vi[k] = want_idx ? fm.part_idx[o] : 0x7fffffff;
      if (!in) { vm[k] = -INFINITY; vl[k] = 0.f; }
    }
  }
  __device__ __forceinline__ StatMerge(const FewMerge& fm, const int32_t* pos_idx, int B, int first, int n, bool write_) : write(write_) {
    lg = n <= 32 ? 5 : n <= 64 ? 6 : n <= 128 ? 7 : 8;
    grps = TH >> lg; row = threadIdx.x & ((1 << lg) - 1); grp = threadIdx.x >> lg;
    i = min(first + row, B - 1); live = first + row < B;
    r = pos_idx[i];
    pt = fm.pos_t[i];   // (whether or not r is valid: no load behind another)
    load(fm, B, grp * FLY);
  }
  // x: 3 TH floats of LDS; lse, pos and, unless null, coeff (2^(t - lse2) - 1 of the positive) take rows 0 .. n2 - 1; rows past
  // the last anchor get +inf / -1 / 0.  Ends with a barrier.
  __device__ __forceinline__ void finish(const FewMerge& fm, int B, int Pn, float* x, float* lse, int* pos, float* coeff) {
    float m = -INFINITY, l = 0.f;
    int idx = 0x7fffffff;
    for (int s0 = grp * FLY; s0 < fm.splits; s0 += grps * FLY) {
      if (s0 != grp * FLY) load(fm, B, s0);
      float mn = m;
#pragma unroll
      for (int k = 0; k < FLY; k++) mn = fmaxf(mn, vm[k]);
      const float ms = mn == -INFINITY ? 0.f : mn;
      l *= ex(m - ms);
#pragma unroll
      for (int k = 0; k < FLY; k++) {
        l += vl[k] * ex(vm[k] - ms);
        if (vm[k] > m || (vm[k] == m && vi[k] < idx)) { m = vm[k]; idx = vi[k]; }
      }
    }
    x[threadIdx.x] = m; x[TH + threadIdx.x] = l; ((int*)x)[2 * TH + threadIdx.x] = idx;
    __syncthreads();
    if (grp == 0) {
      for (int k = 1; k < grps; k++) {
        const int o = (k << lg) + row;
        const float m2 = x[o], l2 = x[TH + o];
        const int i2 = ((int*)x)[2 * TH + o];
        const float mn = fmaxf(m, m2), ms = mn == -INFINITY ? 0.f : mn;
        l = l * ex(m - ms) + l2 * ex(m2 - ms);
        if (m2 > m || (m2 == m && i2 < idx)) idx = i2;
        m = mn;
      }
      const bool ok = r >= 0 && r < Pn;
      const float l2 = m + log2f(l);
      lse[row] = live ? l2 : INFINITY;
      pos[row] = live ? r : -1;
      if (coeff) coeff[row] = live && ok ? exp2f(pt - l2) - 1.f : 0.f;
      if (write && live) {
        fm.lse2[i] = l2;
        fm.rowloss[i] = ok ? (l2 - pt) * kLn2 : NAN;
        if (fm.lse_out) fm.lse_out[i] = l2 * kLn2;
        if (fm.argmax_out) fm.argmax_out[i] = idx;
      }
    }
    __syncthreads();
  }
};
inline FewMerge few_merge_args(const LossArgs& a, const LossPlan& pl) {
  FewMerge fm{};
  fm.splits = pl.stat_splits;
  fm.part_m = (const float*)(a.ws + pl.off_part_m); fm.part_l = (const float*)(a.ws + pl.off_part_l); fm.part_idx = (const int*)(a.ws + pl.off_part_idx);
  fm.pos_t = (const float*)(a.ws + pl.off_pos); fm.lse2 = (float*)(a.ws + pl.off_lse2); fm.rowloss = (float*)(a.ws + pl.off_rowloss);
  fm.lse_out = a.lse; fm.argmax_out = a.argmax;
  return fm;
}
inline StatsSmallArgs stats_small_args(const LossArgs& a, const LossPlan& pl, const unsigned short* q, const unsigned short* p) {
  StatsSmallArgs g{};
  g.Q = q; g.P = p; g.pos_idx = a.pos_idx;
  g.B = a.B; g.Pn = a.P; g.d = a.d; g.n_ablk = (a.B + kStatTile - 1) / kStatTile; g.tiles = (a.P + kStatTile - 1) / kStatTile;
  g.tiles_per_split = pl.stat_cols_per_split / kStatTile; g.mask_self = (a.flags & GC_MASK_SELF) ? 1 : 0;
  g.alpha2 = a.alpha * kLog2e;
  g.part_m = (float*)(a.ws + pl.off_part_m); g.part_l = (float*)(a.ws + pl.off_part_l); g.part_idx = (int*)(a.ws + pl.off_part_idx);
  g.pos_t = (float*)(a.ws + pl.off_pos);
  return g;
}

}  // namespace gc
