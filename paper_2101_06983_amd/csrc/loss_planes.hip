// The loss / representation-gradient path in fp32-grade arithmetic on the bf16 matrix cores: fp32 inputs of any width,
// and bf16 inputs of the widths the kernels of loss_mfma.hip do not take.
//
// Every number that enters a contraction is a sum of bf16 "planes": a stored bf16 value is one plane, an fp32 value is
// three (x = x0 + x1 + x2, each the rounding of what the earlier ones left: 24 bits and more), and so is every softmax
// coefficient.  A product of two sums keeps the pairs (i, j) with i + j <= 2; what is dropped is below 2^-25 of the
// product, less than the rounding of one fp32 operation.  Accumulation is fp32.  fp32 MFMAs would do the same in one
// instruction of 1/16 of the rate: 6 products per pair of fp32 operands cost 6/16 of that, 3 per (coefficient, bf16
// row) 3/16, 1 per pair of bf16 operands 1/16.
//
//   planes_pack_kernel   both inputs into "fragments": 1 KB blocks that hold, in lane order, what a wave loads as one
//                        MFMA operand.  Two copies: contiguous along d (scores) and contiguous along the rows (the
//                        gradient products).  Rows are padded to 128, columns to 64 with zeros, so nothing after this
//                        kernel knows about alignment, odd widths or bounds of its loads.
//   planes_stats_kernel  per anchor: running maximum, sum of 2^t, arg-max, the positive's logit (Eq. 1 / Eq. 4)
//   planes_grad_kernel   Eq. 5 and Eq. 6 in one launch; scores are recomputed, never stored
//
// Layouts (v_mfma_f32_32x32x16_bf16): A lane l holds A[m = l % 32][k = 8 (l / 32) + 0..7], B alike with n, D register r
// of lane l holds D[m = 8 (r / 4) + 4 (l / 32) + r % 4][n = l % 32].  Scores are formed with the streamed rows on M and
// the owner rows on N: registers 8 kk .. 8 kk + 7 of a lane are then one owner row against streamed rows
// 16 kk + {4 h .. 4 h + 3, 8 + 4 h .. 8 + 4 h + 3} (h = l / 32), which is an A fragment of the gradient product for that
// order of the contraction; the row-contiguous copy is packed in the same order.
#include <type_traits>

#include "gc_common.h"
#include "stats_tile.h"

namespace gc {

__device__ __forceinline__ f32x16 mfma_p(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
typedef __attribute__((ext_vector_type(8))) float f32x8_t;

// v as N bf16 planes.  A value that rounds to infinity is truncated instead (so that a finite value stays finite); an
// infinite or NaN value has the one plane and zeros.
// (CHECKED = false: the values are known to be small.)
template <int N, bool CHECKED = true>
__device__ __forceinline__ void to_planes(f32x8_t v, bf16x8 (&out)[N]) {
  out[0] = __builtin_convertvector(v, bf16x8);
  if constexpr (N > 1) {
    f32x8_t h = __builtin_convertvector(out[0], f32x8_t);
    f32x8_t r = v - h;
    // |v| so large that its rounding is infinite, or not finite itself: rare, and r says so (it is not finite then)
    bool odd = false;
#pragma unroll
    for (int e = 0; e < 8; e++) odd |= !(__builtin_fabsf(r[e]) < INFINITY);
    if (CHECKED && odd) {
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const float x = v[e];   // (a bit cast of v[e] itself reads element 0 of the vector)
        if (__builtin_fabsf(r[e]) < INFINITY) continue;
        const bool finite = __builtin_fabsf(x) < INFINITY;
        const float t = finite ? __builtin_bit_cast(float, __builtin_bit_cast(unsigned, x) & 0xffff0000u) : x;
        out[0][e] = (__bf16)t;
        r[e] = finite ? x - t : 0.f;
      }
    }
    out[1] = __builtin_convertvector(r, bf16x8);
    if constexpr (N > 2) out[2] = __builtin_convertvector(r - __builtin_convertvector(out[1], f32x8_t), bf16x8);
  }
}

// ---- pack ------------------------------------------------------------------------------------------------------------
// Fragment blocks of 512 bf16 numbers (64 lanes x 8):
//   xk[((row / 32) * KS + k / 16) * NP + plane]   lane l: row l % 32, k = 16 ks + 8 (l / 32) ..
//   xt[((row / 16) * CT + col / 32) * NP + plane] lane l: column l % 32, rows 16 rs + 4 h + {0..3, 8..11}
struct PackSide { const void* x; unsigned short* xk; unsigned short* xt; int rows, rblocks; };
struct PackArgs { PackSide side[2]; int d, KS, CT, cblocks, nb0; bool vec; };
constexpr int PK_W = 64;   // columns per workgroup
// One workgroup: 32 rows x 64 columns through LDS, a fragment of either copy per wave.  Bound by its loads and stores (one read, two to
// six 16-byte stores per 8 values), in small calls by one trip through them: with 128 columns, half as many workgroups and two fragments
// one after the other, a call takes 48.6 us for 46.9 (512 x 1024 x 1000 bf16), 72.8 for 70.1 (fp32), 49.6 for 47.2 (1024 x 1024 x 200 fp32);
// 2221 for 2218 at 2000 x 16000 x 1000 fp32.
template <typename T>
__global__ void __launch_bounds__(256) planes_pack_kernel(PackArgs a) {
  constexpr int NP = sizeof(T) == 4 ? 3 : 1;
  __shared__ float tile[32][PK_W + 4];
  int id = blockIdx.x;
  const bool second = id >= a.nb0;
  if (second) id -= a.nb0;
  const PackSide s = second ? a.side[1] : a.side[0];
  const int rb = id / a.cblocks, c0 = (id % a.cblocks) * PK_W, r0 = rb * 32;
  const T* x = (const T*)s.x;
  const int tid = threadIdx.x;
  if (a.vec && c0 + PK_W <= a.d) {   // d a multiple of 8 and the base 16-byte aligned: 16-byte loads
    constexpr int E = 16 / sizeof(T), PER_ROW = PK_W / E;
#pragma unroll
    for (int i = 0; i < 32 * PER_ROW / 256; i++) {
      const int q = tid + 256 * i, r = q / PER_ROW, c = (q % PER_ROW) * E;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (r0 + r < s.rows) v = *(const u32x4*)(x + (size_t)(r0 + r) * a.d + c0 + c);
#pragma unroll
      for (int e = 0; e < E; e++) {
        if constexpr (sizeof(T) == 4) tile[r][c + e] = __builtin_bit_cast(f32x4, v)[e];
        else tile[r][c + e] = bf2f((unsigned short)(v[e / 2] >> (16 * (e % 2))));
      }
    }
  } else {
#pragma unroll 4
    for (int i = 0; i < 32 * PK_W / 256; i++) {
      const int q = tid + 256 * i, r = q / PK_W, c = q % PK_W;
      float v = 0.f;
      if (r0 + r < s.rows && c0 + c < a.d) {
        if constexpr (sizeof(T) == 4) v = x[(size_t)(r0 + r) * a.d + c0 + c];
        else v = bf2f(x[(size_t)(r0 + r) * a.d + c0 + c]);
      }
      tile[r][c] = v;
    }
  }
  __syncthreads();
  const int lane = tid & 63, w = tid >> 6, h = lane >> 5, ln = lane & 31;
  {   // 4 k-steps of 16 columns
    const int ks = c0 / 16 + w;
    if (ks < a.KS) {
      f32x8_t v;
#pragma unroll
      for (int e = 0; e < 8; e++) v[e] = tile[ln][16 * w + 8 * h + e];
      bf16x8 p[NP];
      to_planes<NP>(v, p);
#pragma unroll
      for (int n = 0; n < NP; n++) *(bf16x8*)(s.xk + (((size_t)rb * a.KS + ks) * NP + n) * 512 + lane * 8) = p[n];
    }
  }
  {   // 2 row steps x 2 column tiles
    const int i = w >> 1, ct = c0 / 32 + (w & 1);
    if (ct < a.CT) {
      f32x8_t v;
#pragma unroll
      for (int e = 0; e < 8; e++) v[e] = tile[16 * i + 4 * h + (e & 3) + 8 * (e >> 2)][32 * (w & 1) + ln];
      bf16x8 p[NP];
      to_planes<NP>(v, p);
#pragma unroll
      for (int n = 0; n < NP; n++) *(bf16x8*)(s.xt + (((size_t)(2 * rb + i) * a.CT + ct) * NP + n) * 512 + lane * 8) = p[n];
    }
  }
}

// ---- scores ------------------------------------------------------------------------------------------------------------
// An infinite operand, or a product beyond 3.4e38, is an infinity of the right sign in the product of the first planes, but
// times the zeros and the remainders of either sign in the other planes it makes the sum NaN, where an fp32 product is
// +-inf (a target that is masked by such a feature has weight 0).  A tile with a NaN score takes those scores from the
// first planes alone: +-inf or NaN as fp32 arithmetic gives it, since every finite product is lost in the infinite one.
__device__ __forceinline__ bool any_nan(const f32x16& s) {
  bool nan = false;
#pragma unroll
  for (int r = 0; r < 16; r += 2) nan |= __builtin_isunordered(s[r], s[r + 1]);   // either of the two
  return __builtin_amdgcn_ballot_w64(nan) != 0;
}
// (k-steps first, first + step, .. ; str and own point at this lane's piece of fragment 0)
template <int NP>
__device__ __forceinline__ void first_planes_for_nan(const unsigned short* str, const unsigned short* own, int first, int step, int KS, f32x16& s) {
  f32x16 t;
#pragma unroll
  for (int r = 0; r < 16; r++) t[r] = 0.f;
#pragma unroll 4
  for (int ks = first; ks < KS; ks += step)
    t = mfma_p(*(const bf16x8*)(str + (size_t)ks * NP * 512), *(const bf16x8*)(own + (size_t)ks * NP * 512), t);
#pragma unroll
  for (int r = 0; r < 16; r++) s[r] = s[r] != s[r] ? t[r] : s[r];
}

// s[no] += R_tile O_no^T for one 32-row streamed tile (fragments at str, contiguous along k) and NO blocks of 32 owner
// rows: their first ks_lds k-steps are in LDS (own_lds, [k-step][no][plane]), the rest is loaded (own_glb + no * own_stride).
// A wave is alone on its SIMD or with one other, so the latency of L2 is hidden by loads in flight only: PD k-steps ahead,
// 16 KB (12 KB for three planes; with half of that the fp32 call of 512 x 1024 scores at d = 768 took 77 us and not 69).
// k-steps past the end re-read the last one and are not used.
// ks_lds: a multiple of PD, or KS.
constexpr int planes_pd(int NP) { return NP == 1 ? 16 : 4; }
template <int NP, int NO, int PD>
__device__ __forceinline__ void planes_scores(const unsigned short* str, const unsigned short* own_lds, const unsigned short* own_glb,
                                              size_t own_stride, int KS, int ks_lds, f32x16 (&s)[NO]) {
  const int lane = threadIdx.x & 63;
  str += lane * 8; own_lds += lane * 8; own_glb += lane * 8;
  auto products = [&](const bf16x8 (&r)[NP], const bf16x8 (&o)[NP], f32x16& acc) __attribute__((always_inline)) {
#pragma unroll
    for (int t = NP - 1; t >= 0; t--)   // small terms first
#pragma unroll
      for (int i = 0; i <= t; i++) acc = mfma_p(r[i], o[t - i], acc);
  };
  bf16x8 rf[PD][NP];
  auto load_r = [&](int slot, int ks) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NP; n++) rf[slot][n] = *(const bf16x8*)(str + ((size_t)ks * NP + n) * 512);
  };
#pragma unroll
  for (int p = 0; p < PD; p++) load_r(p, min(p, KS - 1));
  for (int k0 = 0; k0 < ks_lds; k0 += PD) {
#pragma unroll
    for (int p = 0; p < PD; p++) {
      const int ks = k0 + p;
      if (ks < ks_lds) {   // uniform; false only behind the last k-step
#pragma unroll
        for (int no = 0; no < NO; no++) {
          bf16x8 o[NP];
#pragma unroll
          for (int n = 0; n < NP; n++) o[n] = *(const bf16x8*)(own_lds + ((ks * NO + no) * NP + n) * 512);
          products(rf[p], o, s[no]);
        }
        load_r(p, min(ks + PD, KS - 1));
      }
    }
  }
  if (ks_lds < KS) {
    constexpr int PO = NP == 1 ? 8 : 2;   // (PD is a multiple: the ring slots of both loops agree)
    bf16x8 of[PO][NO][NP];
    auto load_o = [&](int slot, int ks) __attribute__((always_inline)) {
#pragma unroll
      for (int no = 0; no < NO; no++)
#pragma unroll
        for (int n = 0; n < NP; n++) of[slot][no][n] = *(const bf16x8*)(own_glb + no * own_stride + ((size_t)ks * NP + n) * 512);
    };
#pragma unroll
    for (int p = 0; p < PO; p++) load_o(p, min(ks_lds + p, KS - 1));
    for (int k0 = ks_lds; k0 < KS; k0 += PD) {
#pragma unroll
      for (int p = 0; p < PD; p++) {
        const int ks = k0 + p;
        if (ks < KS) {
#pragma unroll
          for (int no = 0; no < NO; no++) products(rf[p], of[p % PO][no], s[no]);
          load_r(p, min(ks + PD, KS - 1));
          load_o(p % PO, min(ks + PO, KS - 1));
        }
      }
    }
  }
  if constexpr (NP > 1) {
#pragma unroll
    for (int no = 0; no < NO; no++)
      if (any_nan(s[no])) first_planes_for_nan<NP>(str, own_glb + no * own_stride, 0, 1, KS, s[no]);
  }
}

// the first ks_lds k-steps of NO owner blocks into LDS as [k-step][no][plane] blocks of 1 KB
template <int NP, int NO, int THREADS = 256>
__device__ __forceinline__ void planes_stage_own(unsigned short* own_lds, const unsigned short* own_glb, size_t own_stride, int ks_lds) {
  const int per = ks_lds * NP * 64;   // 16-byte pieces per owner block
#pragma unroll
  for (int no = 0; no < NO; no++) {
    const u32x4* src = (const u32x4*)(own_glb + no * own_stride);
    for (int q0 = threadIdx.x; q0 < per; q0 += 8 * THREADS) {   // eight loads in flight
      u32x4 v[8];
#pragma unroll
      for (int i = 0; i < 8; i++) v[i] = src[min(q0 + THREADS * i, per - 1)];
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const int q = q0 + THREADS * i;
        if (q < per) *(u32x4*)(own_lds + ((((q >> 6) / NP) * NO + no) * NP + (q >> 6) % NP) * 512 + (q & 63) * 8) = v[i];
      }
    }
  }
}

// ---- row statistics ------------------------------------------------------------------------------------------------------
struct PlanesStatsArgs {
  const unsigned short* qk; const unsigned short* pk;   // packed along k
  const int32_t* pos_idx;
  int B, P, KS, ks_lds, n_own, tiles, tiles_per_wave;   // tiles: 32-row tiles of the targets
  float alpha2;
  int mask_self;
  float* part_m; float* part_l; int* part_idx; float* pos_t;
};
// A workgroup owns 32 NO anchors; each of its four waves walks target tiles of its own and is a split of its own
// (split = 4 * workgroup split + wave), so that nothing is exchanged between waves.
template <int NP, int NO>
__global__ void __launch_bounds__(256, 2) planes_stats_kernel(PlanesStatsArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned short pl_lds[];
  const int lane = threadIdx.x & 63, h = lane >> 5, ln = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int task = xcd_task_id();
  const int ob = task % g.n_own, split = (task / g.n_own) * 4 + w;
  const size_t blk = (size_t)g.KS * NP * 512;   // one 32-row block
  const unsigned short* own = g.qk + (size_t)ob * NO * blk;
  planes_stage_own<NP, NO>(pl_lds, own, blk, g.ks_lds);
  __syncthreads();
  float m[NO], l[NO], pos[NO];
  int best[NO], r_o[NO], own_idx[NO];
  bool got[NO];
#pragma unroll
  for (int no = 0; no < NO; no++) {
    own_idx[no] = (ob * NO + no) * 32 + ln;
    r_o[no] = own_idx[no] < g.B ? g.pos_idx[own_idx[no]] : -1;
    m[no] = -INFINITY; l[no] = 0.f; pos[no] = 0.f; best[no] = 0x7fffffff; got[no] = false;
  }
  const int t_end = min(g.tiles, (split + 1) * g.tiles_per_wave);
  for (int t = split * g.tiles_per_wave; t < t_end; t++) {
    f32x16 s[NO];
#pragma unroll
    for (int no = 0; no < NO; no++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[no][r] = 0.f;
    planes_scores<NP, NO, planes_pd(NP)>(g.pk + (size_t)t * blk, pl_lds, own, blk, g.KS, g.ks_lds, s);
    const int j0 = t * 32 + 4 * h;   // register r: target j0 + 8 (r / 4) + r % 4, increasing in r
#pragma unroll
    for (int no = 0; no < NO; no++) {
      float mt = -INFINITY;
      int bt = 0x7fffffff;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int j = j0 + 8 * (r >> 2) + (r & 3);
        float v = s[no][r] * g.alpha2;
        const bool masked = j >= g.P || (g.mask_self && j == own_idx[no]);
        if (masked) v = -INFINITY;
        // (a positive that the self-mask removes has the logit -inf: its row loss is then +inf)
        if (j == r_o[no] && j < g.P) { pos[no] = v; got[no] = true; }
        s[no][r] = v;
        if (v > mt) { mt = v; bt = j; }   // strict: the smallest index attaining the maximum
      }
      // a NaN score is never the maximum; it reaches the sum below (and so the loss) through its own term
      const float mn = fmaxf(m[no], mt);
      const float ms = (mn == -INFINITY) ? 0.f : mn;
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; r++) sum += exp2f(s[no][r] - ms);
      l[no] = l[no] * exp2f(m[no] - ms) + sum;
      if (mt > m[no]) best[no] = bt;
      m[no] = mn;
    }
  }
#pragma unroll
  for (int no = 0; no < NO; no++) {
    if (got[no]) g.pos_t[own_idx[no]] = pos[no];   // one lane of one split
    // the other half-wave has the other 16 targets of every tile
    const float m2 = __shfl_xor(m[no], 32), l2 = __shfl_xor(l[no], 32);
    const int b2 = __shfl_xor(best[no], 32);
    const float mn = fmaxf(m[no], m2), ms = (mn == -INFINITY) ? 0.f : mn;
    const float la = h ? l2 : l[no], ma = h ? m2 : m[no], lb = h ? l[no] : l2, mb = h ? m[no] : m2;
    const float ll = la * exp2f(ma - ms) + lb * exp2f(mb - ms);
    const int bi = (m2 > m[no] || (m2 == m[no] && b2 < best[no])) ? b2 : best[no];
    if (h == 0 && own_idx[no] < g.B) {
      const size_t o = (size_t)split * g.B + own_idx[no];
      g.part_m[o] = mn; g.part_l[o] = ll; g.part_idx[o] = bi;
    }
  }
}

// Few scores: 32 x 32 tiles, the k-steps dealt to the four waves of a workgroup, eight (three planes: three) of them in
// flight per wave and nothing staged.  (512 x 1024 scores: fp32 d = 768 11 us, 19.6 with the kernel
// above; bf16 d = 1024 8 us, 12 above.)
template <int NP>
__global__ void __launch_bounds__(256) planes_stats_small_kernel(StatsSmallArgs g, int KS) {
  constexpr int T = kStatTile, PD = NP == 1 ? 8 : 3;
  __shared__ StatTileLds lds;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int task = xcd_task_id();
  const int ob = task % g.n_ablk, split = task / g.n_ablk;
  const size_t blk = (size_t)KS * NP * 512;
  const unsigned short* own = g.Q + (size_t)ob * blk + lane * 8;
  StatTile<true> st(g, ob * T);
  const int t_end = min(g.tiles, (split + 1) * g.tiles_per_split);
  for (int t = split * g.tiles_per_split; t < t_end; t++) {
    const unsigned short* str = g.P + (size_t)t * blk + lane * 8;
    bf16x8 ro[PD][NP], rs[PD][NP];
    auto load = [&](int slot, int ks) __attribute__((always_inline)) {
#pragma unroll
      for (int n = 0; n < NP; n++) {
        rs[slot][n] = *(const bf16x8*)(str + ((size_t)ks * NP + n) * 512);
        ro[slot][n] = *(const bf16x8*)(own + ((size_t)ks * NP + n) * 512);
      }
    };
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.f;
#pragma unroll
    for (int p = 0; p < PD; p++) load(p, min(wave + 4 * p, KS - 1));
    for (int k0 = wave; k0 < KS; k0 += 4 * PD) {
#pragma unroll
      for (int p = 0; p < PD; p++) {
        const int ks = k0 + 4 * p;
        if (ks < KS) {
#pragma unroll
          for (int x = NP - 1; x >= 0; x--)   // small terms first
#pragma unroll
            for (int i = 0; i <= x; i++) acc = mfma_p(rs[p][i], ro[p][x - i], acc);
          load(p, min(ks + 4 * PD, KS - 1));
        }
      }
    }
    if constexpr (NP > 1)
      if (any_nan(acc)) first_planes_for_nan<NP>(str, own, wave, 4, KS, acc);
    StatTile<true>::put(lds, wave, acc);
    __syncthreads();
    st.tile(g, lds, t * T);
    __syncthreads();   // the partial tiles have been read
  }
  st.finish(g, lds, split);
}

// ---- gradients -----------------------------------------------------------------------------------------------------------
// A workgroup owns 32 NO rows and up to 128 CTW columns of dQ (or dP) and walks a range of the other side 128 rows at a
// time.  Per step each wave forms the scores of 32 of those rows against the owner rows over the whole width, turns them
// into coefficients g = 2^(t - lse2) - [j = r_i] (fp32, Eq. 5 / Eq. 6) and publishes them as three bf16 planes of
// ready-made A fragments; then every wave multiplies all 128 rows' coefficients with its own column tiles (w, w + 4, ..).
// The positive's coefficient comes from the statistics' own sum of its score, the one that is part of lse2: where the softmax
// has converged on it, the rounding of a second sum would be most of the coefficient (5.7e-5 of dq at 512 x 1024 x 776 and
// temperature 0.1, 4.2e-6 so).
// (Registers spilled: 30 by <1, 2, 8>, bf16 of 769 to 1024 columns with 64 owner rows; none by the others.)
struct PlanesRole {
  const unsigned short* own_k; const unsigned short* str_k; const unsigned short* str_t;
  int n_own, n_str;         // valid rows
  int oblk, splits, len;    // owner blocks, splits of the streamed rows, rows per split (a multiple of 128)
  float* out; size_t split_stride;
};
struct PlanesGradArgs {
  PlanesRole role[2];       // 0: owner = anchors (dQ), 1: owner = targets (dP)
  int n0;                   // workgroups of role 0
  int d, KS, CT, ks_lds, col_slices, ct_per_slice;
  const float* lse2; const int32_t* pos;   // per anchor, padded to 128 rows with +inf / -1
  const float* pos_c;                      // ... the positive's coefficient, with room for 128 rows
  float alpha2, out_scale;
  int mask_self;
  FewMerge fm; int P;                      // MERGE: lse2, pos (not padded) and pos_c are formed from these
};
constexpr int PG_STEP = 128, PG_MERGE_BYTES = 3 * kFewMergeRows * 4;
constexpr int planes_g_bytes(int NO) { return 4 * 2 * 3 * NO * 1024; }
// Widths of more than 512 columns with 32 owner rows: the workgroup is alone on its compute unit (LDS, accumulators), and its time
// is that of its loads from L2.  Eight waves, two to a SIMD, have twice as many of them in flight: waves w and w + 4 form half of the
// k-steps each of the same scores, meet in LDS, finish half of the coefficients each and own half of the columns each.  (A call with
// four and with eight waves: 59.9 and 55.9 us at 512 x 1024 x 768 in fp32, 48.0 and 45.2 at x 1024 in bf16.  With 64 owner rows the
// accumulators of half of the columns are too many registers for two waves; up to 512 columns two workgroups share a compute unit.)
constexpr int planes_g_waves(int NO, int CTW) { return CTW > 4 && NO == 1 ? 8 : 4; }

// MERGE: the statistics come as splits, see StatMerge (a template argument: as a branch at run time it costs the instantiations
// that never take it registers, and <3, 2, 8> seven spills inside its loop; 58.9 us a call at 512 x 1024 x 768 in fp32, 57.7 so).
template <int NP, int NO, int CTW, bool MERGE>
__global__ void __launch_bounds__(64 * planes_g_waves(NO, CTW), planes_g_waves(NO, CTW) == 8 || (NO == 1 && CTW <= 4) ? 2 : 1)
planes_grad_kernel(PlanesGradArgs g) {
  constexpr int NW = planes_g_waves(NO, CTW), NH = NW / 4, CW = CTW / NH;   // halves of the k-steps; column tiles of a wave
  extern __shared__ __attribute__((aligned(16))) unsigned short pl_lds[];
  unsigned short* gl = pl_lds;                                    // [kk8][no][plane] blocks of 1 KB
  unsigned short* own_lds = pl_lds + planes_g_bytes(NO) / 2;
  const int lane = threadIdx.x & 63, h = lane >> 5, ln = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), wr = w & 3, wh = w >> 2;   // rows and half of the k-steps
  int k0 = 0, k1 = g.KS;
  if constexpr (NH == 2) {   // (whole turns of the ring of planes_scores where LDS does not hold every k-step of the owner rows)
    constexpr int PD = planes_pd(NP);
    const int km = g.ks_lds == g.KS ? g.KS / 2 : (g.KS / 2 + PD / 2) / PD * PD;
    if (wh) k0 = km; else k1 = km;
  }
  int id = xcd_task_id();
  const int ri = id >= g.n0 ? 1 : 0;
  if (ri) id -= g.n0;
  const PlanesRole R = ri ? g.role[1] : g.role[0];
  const int ob = id % R.oblk, cs = (id / R.oblk) % g.col_slices, split = id / (R.oblk * g.col_slices);
  const size_t blk = (size_t)g.KS * NP * 512;
  const unsigned short* own = R.own_k + (size_t)ob * NO * blk;
  const int sbeg = split * R.len, send = min(R.n_str, sbeg + R.len);
  const int ct0 = cs * g.ct_per_slice, ct1 = min(g.CT, ct0 + g.ct_per_slice);
  float* const l_lse = (float*)(own_lds + (size_t)g.ks_lds * NO * NP * 512);   // (MERGE) of rows from the first owner / streamed row on
  int* const l_pos = (int*)l_lse + kFewMergeRows;
  float* const l_c = l_lse + 2 * kFewMergeRows;
  if constexpr (MERGE) {
    const int B = ri ? R.n_str : R.n_own;
    StatMerge<true, 64 * NW> sm(g.fm, g.pos, B, ri ? sbeg : ob * NO * 32, ri ? send - sbeg : NO * 32, !ri && split == 0 && cs == 0);
    planes_stage_own<NP, NO, 64 * NW>(own_lds, own, blk, g.ks_lds);
    sm.finish(g.fm, B, g.P, (float*)gl, l_lse, l_pos, l_c);
  } else {
    planes_stage_own<NP, NO, 64 * NW>(own_lds, own, blk, g.ks_lds);
  }

  int own_idx[NO], r_o[NO];
  float lse_o[NO], c_o[NO];
#pragma unroll
  for (int no = 0; no < NO; no++) {
    own_idx[no] = (ob * NO + no) * 32 + ln;
    lse_o[no] = ri ? 0.f : MERGE ? l_lse[no * 32 + ln] : g.lse2[own_idx[no]];
    c_o[no] = ri ? 0.f : MERGE ? l_c[no * 32 + ln] : g.pos_c[own_idx[no]];
    r_o[no] = ri ? -1 : MERGE ? l_pos[no * 32 + ln] : g.pos[own_idx[no]];
  }
  f32x16 acc[NO][CW];
#pragma unroll
  for (int no = 0; no < NO; no++)
#pragma unroll
    for (int i = 0; i < CW; i++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[no][i][r] = 0.f;
  __syncthreads();

  for (int t0 = sbeg; t0 < send; t0 += PG_STEP) {
    // scores of streamed rows t0 + 32 wr .. + 31, k-steps k0 .. k1 - 1
    f32x16 s[NO];
#pragma unroll
    for (int no = 0; no < NO; no++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[no][r] = 0.f;
    planes_scores<NP, NO, planes_pd(NP)>(R.str_k + (size_t)(t0 / 32 + wr) * blk + k0 * NP * 512, own_lds + k0 * NO * NP * 512, own + k0 * NP * 512,
                                         blk, k1 - k0, min(max(g.ks_lds - k0, 0), k1 - k0), s);
    // the first loads of the second contraction
    constexpr int MOST = NP == 1 ? 16 : CW >= 6 ? 5 : 6, XD = 8 * CW < MOST ? 8 * CW : MOST;   // column tiles in flight
    const unsigned short* xt = R.str_t + (size_t)(t0 / 16) * g.CT * NP * 512 + lane * 8;
    bf16x8 xf[XD][NP];
    auto load_x = [&](int slot, int kk, int i) __attribute__((always_inline)) {
      const unsigned short* p = xt + ((size_t)kk * g.CT + min(ct0 + w + NW * i, g.CT - 1)) * (NP * 512);
#pragma unroll
      for (int n = 0; n < NP; n++) xf[slot][n] = *(const bf16x8*)(p + n * 512);
    };
#pragma unroll
    for (int p = 0; p < XD; p++) load_x(p, p / CW, p % CW);
    const int j0 = t0 + 32 * wr + 4 * h;
    constexpr int NS = 16 / NH;   // scores of this lane: NH = 2: registers 8 wh .. 8 wh + 7, both halves of the sum
    const int rq = NH == 2 ? 16 * wh : 0;   // their first streamed row beyond j0
    if constexpr (NH == 2) {
      // The other half's registers go to where that wave puts its coefficients, which is behind its reads.
      f32x4* mine = (f32x4*)(gl + (2 * wr + wh) * 3 * 512) + lane;
      f32x4* other = (f32x4*)(gl + (2 * wr + 1 - wh) * 3 * 512) + lane;
      f32x4 t[2];
#pragma unroll
      for (int r = 0; r < 8; r++) {
        t[r / 4][r % 4] = wh ? s[0][r] : s[0][8 + r];
        s[0][r] = wh ? s[0][8 + r] : s[0][r];
      }
      other[0] = t[0]; other[64] = t[1];
      __syncthreads();
      t[0] = mine[0]; t[1] = mine[64];
#pragma unroll
      for (int r = 0; r < 8; r++) s[0][r] += t[r / 4][r % 4];
    }
    float lse_s[NS], c_s[NS]; int pos_s[NS];
    if (ri) {
#pragma unroll
      for (int q = 0; q < NS / 4; q++) {
        f32x4 a, c;
        i32x4 b;
        if constexpr (MERGE) {
          const int o = j0 + rq - sbeg + 8 * q;
          a = *(const f32x4*)(l_lse + o); b = *(const i32x4*)(l_pos + o); c = *(const f32x4*)(l_c + o);
        } else {
          const int o = j0 + rq + 8 * q;
          a = *(const f32x4*)(g.lse2 + o); b = *(const i32x4*)(g.pos + o); c = *(const f32x4*)(g.pos_c + o);
        }
#pragma unroll
        for (int e = 0; e < 4; e++) { lse_s[4 * q + e] = a[e]; pos_s[4 * q + e] = b[e]; c_s[4 * q + e] = c[e]; }
      }
    }
#pragma unroll
    for (int no = 0; no < NO; no++) {
#pragma unroll
      for (int r = 0; r < NS; r++) {
        const int j = j0 + rq + 8 * (r >> 2) + (r & 3);
        const float lse = ri ? lse_s[r] : lse_o[no];
        const bool hit = ri ? pos_s[r] == own_idx[no] : r_o[no] == j;
        float v = hit ? (ri ? c_s[r] : c_o[no]) : exp2f(s[no][r] * g.alpha2 - lse);
        if (j >= R.n_str || (g.mask_self && j == own_idx[no])) v = 0.f;
        s[no][r] = v;
      }
#pragma unroll
      for (int kk = 0; kk < NS / 8; kk++) {
        f32x8_t v;
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = s[no][8 * kk + e];
        bf16x8 p[3];
        to_planes<3, false>(v, p);
#pragma unroll
        for (int n = 0; n < 3; n++) *(bf16x8*)(gl + (((2 * wr + wh + kk) * NO + no) * 3 + n) * 512 + lane * 8) = p[n];
      }
    }
    __syncthreads();
    // dO[32 NO x columns] += g[32 NO x 128] R[128 x columns]; the row blocks of the packed copy are full (zero-padded).
    // The first loads have been issued before the coefficients were formed; the coefficients come a row step ahead.
    bf16x8 gf[2][NO][3];
    auto load_g = [&](int slot, int kk) __attribute__((always_inline)) {
#pragma unroll
      for (int no = 0; no < NO; no++)
#pragma unroll
        for (int n = 0; n < 3; n++) gf[slot][no][n] = *(const bf16x8*)(gl + ((kk * NO + no) * 3 + n) * 512 + lane * 8);
    };
    load_g(0, 0);
#pragma unroll
    for (int kk = 0; kk < 8; kk++) {
      if (kk < 7) load_g((kk + 1) & 1, kk + 1);
#pragma unroll
      for (int i = 0; i < CW; i++) {
        constexpr int N = 8 * CW;
        const int at = kk * CW + i;
        bf16x8 x[NP];
#pragma unroll
        for (int n = 0; n < NP; n++) x[n] = xf[at % XD][n];
        if (at + XD < N) load_x(at % XD, (at + XD) / CW, (at + XD) % CW);
        if (ct0 + w + NW * i < ct1) {
#pragma unroll
          for (int no = 0; no < NO; no++)
#pragma unroll
            for (int t = 2; t >= 0; t--)
#pragma unroll
              for (int n = 0; n < NP; n++)
                if (t - n >= 0) acc[no][i] = mfma_p(gf[kk & 1][no][t - n], x[n], acc[no][i]);
        }
      }
    }
    __syncthreads();   // the coefficients have been read: the next step may overwrite them
  }

  float* out = R.out + (size_t)split * R.split_stride;
#pragma unroll
  for (int i = 0; i < CW; i++) {
    const int ct = ct0 + w + NW * i, col = 32 * ct + ln;
    if (ct < ct1 && col < g.d) {
#pragma unroll
      for (int no = 0; no < NO; no++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int row = (ob * NO + no) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
          if (row < R.n_own) out[(size_t)row * g.d + col] = acc[no][i][r] * g.out_scale;
        }
    }
  }
}

// ---- host ------------------------------------------------------------------------------------------------------------
static inline int cdiv(int a, int b) { return (a + b - 1) / b; }
static inline int pad_to(int a, int b) { return cdiv(a, b) * b; }

// Fills the planes part of a plan (sizes in rows and bytes; make_loss_plan lays the workspace out).
void plan_planes(LossPlan& pl, int B, int P, int d, gc_dtype dt, int max_splits) {
  const int cu = num_cu();
  pl.np = dt == GC_F32 ? 3 : 1;
  const int dpad = pad_to(d, 64);
  pl.px_KS = dpad / 16; pl.px_CT = dpad / 32;
  pl.px_rows_q = pad_to(B, 128); pl.px_rows_p = pad_to(P, 128);
  const int tiles = cdiv(P, 32);
  if ((long long)B * P <= (1ll << 20)) {   // few scores: small tiles (the line of the bf16 widths, see stats_small_kernel)
    pl.stat_tile = kStatTile;
    const int per = cdiv(tiles, 64);       // the merge kernel combines at most 64 splits
    pl.stat_cols_per_split = per * kStatTile;
    pl.stat_splits = cdiv(tiles, per);
  } else {   // about eight waves for every CU, each wave a split of its own
    int wgs = cdiv(2 * cu, cdiv(B, 32));
    if (wgs > 16) wgs = 16;
    if (wgs > cdiv(tiles, 4)) wgs = cdiv(tiles, 4);
    pl.px_tiles_per_wave = cdiv(tiles, 4 * wgs);
    pl.stat_splits = 4 * cdiv(tiles, 4 * pl.px_tiles_per_wave);
  }
  // gradients
  pl.px_col_slices = cdiv(pl.px_CT, 32);                       // a workgroup holds up to 1024 columns
  pl.px_ct_per_slice = cdiv(pl.px_CT, pl.px_col_slices);
  const int stQ = cdiv(P, PG_STEP), stP = cdiv(B, PG_STEP);    // steps of a whole stream
  auto units = [&](int no) { return (long long)pl.px_col_slices * ((long long)cdiv(B, 32 * no) * stQ + (long long)cdiv(P, 32 * no) * stP); };
  pl.px_no = units(2) >= 8ll * cu ? 2 : 1;
  const long long want = pl.px_no == 1 && pl.px_ct_per_slice <= 16 ? 2 * cu : cu;   // workgroups that run at once
  long long per = (units(pl.px_no) + want - 1) / want;
  if (per < 1) per = 1;
  auto split_of = [&](int steps, int rows, int& ns, int& len) {
    ns = (int)((steps + per - 1) / per);
    if (ns > max_splits) ns = max_splits;
    len = cdiv(steps, ns) * PG_STEP;
    ns = cdiv(rows, len);
  };
  split_of(stQ, P, pl.nsq, pl.q_stream_len);
  split_of(stP, B, pl.nsp, pl.p_stream_len);
  // (64 owner rows are for many steps a workgroup, where a launch more is nothing: no instantiations of their own)
  pl.few_merge = pl.stat_tile && pl.px_no == 1 && pl.p_stream_len <= kFewMergeRows && pl.p_stream_len * pl.stat_splits <= kFewMergeEntries;
}

template <typename T>
static hipError_t pack_t(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws2;
  PackArgs g{};
  g.side[0] = {a.q, (unsigned short*)(ws + pl.off_qk), (unsigned short*)(ws + pl.off_qt), a.B, pl.px_rows_q / 32};
  g.side[1] = {a.p, (unsigned short*)(ws + pl.off_pk), (unsigned short*)(ws + pl.off_pt), a.P, pl.px_rows_p / 32};
  g.d = a.d; g.KS = pl.px_KS; g.CT = pl.px_CT; g.cblocks = cdiv(pl.px_KS * 16, PK_W);
  g.nb0 = g.side[0].rblocks * g.cblocks;
  g.vec = a.d % 8 == 0 && (((uintptr_t)a.q | (uintptr_t)a.p) & 15) == 0;
  planes_pack_kernel<T><<<g.nb0 + g.side[1].rblocks * g.cblocks, 256, 0, a.stream>>>(g);
  return hipGetLastError();
}

// k-steps of the owner rows that LDS holds, of `room`: all, or whole turns of the ring of planes_scores
static int ks_in_lds(int room, int KS, int pd) { return room >= KS ? KS : room / pd * pd; }

template <int NP>
static hipError_t stats_np(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  if (pl.stat_tile) {
    const StatsSmallArgs g = stats_small_args(a, pl, (const unsigned short*)(a.ws2 + pl.off_qk), (const unsigned short*)(a.ws2 + pl.off_pk));
    planes_stats_small_kernel<NP><<<g.n_ablk * pl.stat_splits, 256, 0, a.stream>>>(g, pl.px_KS);
    return hipGetLastError();
  }
  PlanesStatsArgs g{};
  g.qk = (const unsigned short*)(a.ws2 + pl.off_qk); g.pk = (const unsigned short*)(a.ws2 + pl.off_pk);
  g.pos_idx = a.pos_idx; g.B = a.B; g.P = a.P; g.KS = pl.px_KS;
  g.n_own = cdiv(a.B, 32); g.tiles = cdiv(a.P, 32); g.tiles_per_wave = pl.px_tiles_per_wave;
  g.alpha2 = a.alpha * kLog2e; g.mask_self = (a.flags & GC_MASK_SELF) ? 1 : 0;
  g.part_m = (float*)(ws + pl.off_part_m); g.part_l = (float*)(ws + pl.off_part_l); g.part_idx = (int*)(ws + pl.off_part_idx);
  g.pos_t = (float*)(ws + pl.off_pos);
  const int nwg = g.n_own * (pl.stat_splits / 4);
  const int budget = (nwg <= num_cu() ? 152 : 76) * 1024;
  g.ks_lds = ks_in_lds(budget / (NP * 1024), g.KS, planes_pd(NP));
  static bool done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)planes_stats_kernel<NP, 1>, 160 * 1024, done); e != hipSuccess) return e;
  planes_stats_kernel<NP, 1><<<nwg, 256, g.ks_lds * NP * 1024, a.stream>>>(g);
  return hipGetLastError();
}

hipError_t launch_stats_planes(const LossArgs& a, const LossPlan& pl) {
  const hipError_t e = a.dt == GC_F32 ? pack_t<float>(a, pl) : pack_t<unsigned short>(a, pl);
  if (e != hipSuccess) return e;
  return pl.np == 3 ? stats_np<3>(a, pl) : stats_np<1>(a, pl);
}

template <int NP, int NO, int CTW, bool MERGE>
static hipError_t grad_launch_as(PlanesGradArgs& g, int nwg, hipStream_t s) {
  constexpr int merge = MERGE ? PG_MERGE_BYTES : 0;
  const int budget = ((nwg <= num_cu() || NO == 2 || CTW > 4) ? 156 : 78) * 1024 - planes_g_bytes(NO) - merge;
  g.ks_lds = ks_in_lds(budget / (NO * NP * 1024), g.KS, planes_pd(NP));
  static bool done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)planes_grad_kernel<NP, NO, CTW, MERGE>, 160 * 1024, done); e != hipSuccess) return e;
  planes_grad_kernel<NP, NO, CTW, MERGE><<<nwg, 64 * planes_g_waves(NO, CTW), planes_g_bytes(NO) + g.ks_lds * NO * NP * 1024 + merge, s>>>(g);
  return hipGetLastError();
}
template <int NP, int NO, int CTW>
static hipError_t grad_launch(PlanesGradArgs& g, int nwg, hipStream_t s) {
  if constexpr (NO == 1) {   // (few_merge: plan_planes)
    if (g.fm.splits) return grad_launch_as<NP, NO, CTW, true>(g, nwg, s);
  }
  return grad_launch_as<NP, NO, CTW, false>(g, nwg, s);
}
template <int NP, int NO>
static hipError_t grad_ctw(PlanesGradArgs& g, int nwg, hipStream_t s) {
  const int ctw = cdiv(g.ct_per_slice, 4);
  if (ctw <= 1) return grad_launch<NP, NO, 1>(g, nwg, s);
  if (ctw <= 2) return grad_launch<NP, NO, 2>(g, nwg, s);
  if (ctw <= 4) return grad_launch<NP, NO, 4>(g, nwg, s);
  if (ctw <= 6) return grad_launch<NP, NO, 6>(g, nwg, s);
  return grad_launch<NP, NO, 8>(g, nwg, s);
}

hipError_t launch_grad_planes(const LossArgs& a, const LossPlan& pl) {
  char* ws = a.ws;
  auto at = [&](size_t off) { return (const unsigned short*)(a.ws2 + off); };
  PlanesGradArgs g{};
  g.d = a.d; g.KS = pl.px_KS; g.CT = pl.px_CT; g.col_slices = pl.px_col_slices; g.ct_per_slice = pl.px_ct_per_slice;
  g.lse2 = (const float*)(ws + pl.off_lse2); g.pos = (const int32_t*)(ws + pl.off_pos_pad); g.pos_c = (const float*)(ws + pl.off_pos);
  g.alpha2 = a.alpha * kLog2e; g.out_scale = a.alpha / (float)a.B * (a.grad_mul != 0.f ? a.grad_mul : 1.f);
  g.mask_self = (a.flags & GC_MASK_SELF) ? 1 : 0;
  if (merges_itself(a, pl)) { g.fm = few_merge_args(a, pl); g.pos = a.pos_idx; g.P = a.P; }
  const bool want_q = a.dq || a.dz, want_p = a.dp || a.dz;
  const int own = 32 * pl.px_no;
  // a single split writes the result itself, several (and the two halves of dz) leave partials
  float* part_q = (float*)(a.ws2 + pl.off_dq_part);
  float* part_p = (float*)(a.ws2 + pl.off_dp_part);
  const bool direct_q = a.dq && !a.dz && pl.nsq == 1, direct_p = a.dp && !a.dz && pl.nsp == 1;
  g.role[0] = {at(pl.off_qk), at(pl.off_pk), at(pl.off_pt), a.B, a.P, want_q ? cdiv(a.B, own) : 0, pl.nsq, pl.q_stream_len,
               direct_q ? a.dq : part_q, pl.px_stride_q};
  g.role[1] = {at(pl.off_pk), at(pl.off_qk), at(pl.off_qt), a.P, a.B, want_p ? cdiv(a.P, own) : 0, pl.nsp, pl.p_stream_len,
               direct_p ? a.dp : part_p, pl.px_stride_p};
  g.n0 = g.role[0].oblk * pl.nsq * g.col_slices;
  const int nwg = g.n0 + g.role[1].oblk * pl.nsp * g.col_slices;
  hipError_t e = hipSuccess;
  if (pl.np == 3) e = pl.px_no == 2 ? grad_ctw<3, 2>(g, nwg, a.stream) : grad_ctw<3, 1>(g, nwg, a.stream);
  else e = pl.px_no == 2 ? grad_ctw<1, 2>(g, nwg, a.stream) : grad_ctw<1, 1>(g, nwg, a.stream);
  if (e != hipSuccess) return e;
  prof_mark_grad_kernel_done(a.stream);
  // fixed-order sums of the partials; the launch also sums the row losses
  ReduceJob job[2] = {};
  int n = 0;
  auto add = [&](float* out, int rows, const float* part, int count, size_t stride) {
    ReduceJob& j = job[n++];
    j.out = out; j.n = (size_t)rows * a.d; j.nsrc = 1; j.ptr[0] = part; j.count[0] = count; j.stride[0] = stride;
  };
  if (a.dz) {   // both roles' partials into one output
    add(a.dz, a.B, part_q, pl.nsq, pl.px_stride_q);
    job[0].nsrc = 2; job[0].ptr[1] = part_p; job[0].count[1] = pl.nsp; job[0].stride[1] = pl.px_stride_p;
  } else {
    if (a.dq && !direct_q) add(a.dq, a.B, part_q, pl.nsq, pl.px_stride_q);
    if (a.dp && !direct_p) add(a.dp, a.P, part_p, pl.nsp, pl.px_stride_p);
  }
  return launch_reduce_jobs(job, n, a.stream, a.loss_with_partials ? &a : nullptr, &pl);
}

}  // namespace gc
