// Gradient pass of the bf16 loss path for few scores (gfx950; widths that are multiples of 128 up to 768).
#include "mfma_common.h"

namespace gc {

// ===========================================================================
// What the walks of loss_mfma.hip do (a wave keeps its D/4-column slice of the owner rows in registers, only ever touches the
// same columns of the streamed tiles, and the four partial score tiles meet in LDS), in a form for calls whose walks are a few
// tiles long: 32 owner rows and 32 streamed rows a step, no unrolling over stages or waves.  The long form takes 14 us before
// it has done anything (15 us for 2 workgroups of a 64 x 64 problem): its 60 KB of code, of which a short walk runs every
// instruction once, come out of L2 line by line.  Per step: 12 + 12 MFMAs a wave at d = 768 and two barriers.
// ===========================================================================
constexpr int GF_OWN = kFewOwn, GF_T = 32, GF_STAGES = 3;

template <int D, bool MERGE>
struct FewCfg {
  static constexpr int DS = D / 4;               // columns per wave
  static constexpr int KS = DS / 16, CT = DS / 32;   // MFMA k-steps of phase 1, column tiles of phase 2
  static constexpr int C16 = DS / 8;             // 16-byte chunks per slice row
  static constexpr bool SWZ = (C16 % 16) == 8;   // rows of chunks swizzled by row bits, else one pad chunk per row (as in the walks)
  static constexpr int SLOTS = SWZ ? C16 : C16 + 1;
  static constexpr int LDB = SLOTS * 16;
  static constexpr int NI = (GF_T * SLOTS + 63) / 64;   // direct-to-LDS load instructions per tile slice
  // the (row, chunk) pattern of the loads repeats after NP of them, NROWS rows on (swizzled rows; else every load has its own)
  static constexpr int NP = !SWZ ? NI : SLOTS == 24 ? 3 : 1, NROWS = 64 * NP / SLOTS;
  static_assert(!SWZ || (NP * 64 == NROWS * SLOTS && NROWS % 8 == 0 && NI % NP == 0), "pattern of the loads");
  static constexpr int TOFF = MERGE ? 0 : 128;   // a stage starts with lse and pos_idx of the 8 streamed rows this wave finishes
  static constexpr int STAGE = TOFF + NI * 1024;
  static constexpr int X_OFF = 4 * GF_STAGES * STAGE, X_BYTES = 4 * 3 * 1024;   // partial scores [dst wave][src wave ^ dst - 1]
  static constexpr int G_OFF = X_OFF + X_BYTES, L_OFF = G_OFF + 2 * 1024;       // coefficients as A fragments [k-step]
  static constexpr int SMEM = L_OFF + (MERGE ? 2 * kFewMergeRows * 4 : 0);      // merged lse2, and pos_idx, of the rows that need one
  static_assert(SMEM <= 160 * 1024, "LDS budget");
  static_assert(GF_OWN == 32, "a wave's owner rows are one MFMA tile");
};
__device__ __forceinline__ int few_swz(int row) { return (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1); }

// MERGE: the statistics come as splits, see StatMerge.
template <int D, bool OWNER_IS_Q, bool SYM, bool MERGE>
__device__ __forceinline__ void grad_few_body(const GradArgs& ga, const FewMerge& fm, int oblk, int split, unsigned char* smem) {
  using C = FewCfg<D, MERGE>;
  constexpr bool STR_STATS = (SYM || !OWNER_IS_Q) && !MERGE;   // they ride in the stage
  bool one_exp = false;   // see kWideLse
  if constexpr (SYM) one_exp = __builtin_amdgcn_readfirstlane(*ga.wide) == 0;
  const float* stat_q = SYM && one_exp ? ga.wexp : ga.lse2;
  const float* stat_p = SYM && one_exp ? ga.wexp_t : ga.lse2_t;
  const float* lse_own = (SYM && !OWNER_IS_Q) ? stat_p : stat_q;
  const float* lse_str = (SYM && OWNER_IS_Q) ? stat_p : stat_q;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 5, ln = lane & 31;
  const int l16 = lane & 15, g16 = lane >> 4;
  const unsigned short* O = OWNER_IS_Q ? ga.Q : ga.P;
  const unsigned short* R = OWNER_IS_Q ? ga.P : ga.Q;
  const int No = OWNER_IS_Q ? ga.B : ga.Pn, Nr = OWNER_IS_Q ? ga.Pn : ga.B;
  const int slen = OWNER_IS_Q ? ga.q_stream_len : ga.p_stream_len;
  const int a0 = oblk * GF_OWN;
  const int sbeg = split * slen, send = min(Nr, sbeg + slen);
  const int nt = (send - sbeg + GF_T - 1) / GF_T;   // >= 1

  // ---- direct-to-LDS loads of a tile slice: slot q = it * 64 + lane -> (row, chunk) -----------------------------------
  const unsigned ring = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)smem) + w * GF_STAGES * C::STAGE;
  auto slot_src = [&](int it, int max_row) __attribute__((always_inline)) -> unsigned {
    const int q = it * 64 + lane, row = min(min(q / C::SLOTS, GF_T - 1), max_row);
    int c = min(q % C::SLOTS, C::C16 - 1);
    if (C::SWZ) c ^= few_swz(row);
    return (unsigned)((row * D + w * C::DS + c * 8) * 2);
  };
  unsigned src_off[C::NP];
#pragma unroll
  for (int it = 0; it < C::NP; it++) src_off[it] = slot_src(it, GF_T - 1);
  // lanes 0-1 load lse_str of rows 8 w .. 8 w + 7 of the tile, lanes 2-3 pos_pad (dP role)
  const unsigned ri_off = 32u * w + 16u * (lane & 1) + ((lane & 2) && !OWNER_IS_Q ? (unsigned)((const char*)ga.pos_pad - (const char*)lse_str) : 0u);
  auto prefetch = [&](int u, int stage) __attribute__((always_inline)) {
    const int t0 = sbeg + u * GF_T;
    const unsigned short* tile = R + (size_t)t0 * D;
    const unsigned lds = ring + stage * C::STAGE;
    if (STR_STATS && lane < 4) dma_piece<0>(lse_str + t0, ri_off, lds);
    if (t0 + GF_T <= Nr) {
#pragma unroll
      for (int it = 0; it < C::NI; it++) dma_group<1>(tile + (it / C::NP) * C::NROWS * D, &src_off[it % C::NP], lds + C::TOFF + it * 1024);
    } else {   // rows past the end re-read the last valid row (their coefficients are forced to 0)
#pragma unroll 1
      for (int it = 0; it < C::NI; it++) {
        const unsigned off = slot_src(it, Nr - 1 - t0);
        dma_group<1>(tile, &off, lds + C::TOFF + it * 1024);
      }
    }
  };
  SharedCheck chk(ga);
  for (int u = 0; u < min(nt, GF_STAGES); u++) prefetch(u, u);

  // owner slice as phase-1 B fragments: lane (ln, h) holds owner row ln, columns w DS + 16 ks + 8 h .. + 7
  bf16x8 ofrag[C::KS];
  {
    const int row = min(a0 + ln, No - 1);
#pragma unroll
    for (int ks = 0; ks < C::KS; ks++) ofrag[ks] = *(const bf16x8*)(O + (size_t)row * D + w * C::DS + 16 * ks + 8 * h);
  }
  const int a_q = a0 + ln;
  float lse_a = 0.f;
  int r_a = -1;
  if (a_q < No) {
    if ((OWNER_IS_Q || SYM) && !MERGE) lse_a = lse_own[a_q];
    if (OWNER_IS_Q) r_a = ga.pos_pad[a_q];
  }
  float* const lds_lse = (float*)(smem + C::L_OFF);
  int* const lds_pos = (int*)(smem + C::L_OFF) + kFewMergeRows;
  if constexpr (MERGE) {
    StatMerge<false> sm(fm, ga.pos_pad, ga.B, OWNER_IS_Q ? a0 : sbeg, OWNER_IS_Q ? GF_OWN : send - sbeg, OWNER_IS_Q && split == 0);
    sm.finish(fm, ga.B, ga.Pn, (float*)(smem + C::X_OFF), lds_lse, lds_pos, nullptr);   // (the partial scores are not there yet)
    if (OWNER_IS_Q) lse_a = lds_lse[ln];
  }
#pragma unroll
  for (int ks = 0; ks < C::KS; ks++) asm volatile("" : "+v"(ofrag[ks]));   // the compiler's own loads end here
  asm volatile("" : "+v"(lse_a), "+v"(r_a));
  chk.look(ga);

  // per-lane LDS addresses (see lane_base of the walks): + stage, + 64 i for chunk 4 i + j
  auto lane_base = [&](int row, int j, int parity) __attribute__((always_inline)) -> unsigned {
    const int sw = C::SWZ ? few_swz(row) : 0, s2 = sw >> 2, s01 = sw & 3;
    return w * GF_STAGES * C::STAGE + C::TOFF + (unsigned)(row * C::LDB + 16 * (j ^ s01) + (parity ? -64 * s2 : 64 * s2));
  };
  // phase 1: row ln, chunk 2 ks + h = 4 (ks / 2) + 2 (ks & 1) + h
  unsigned p1[2][2], p2lo[2], p2hi[2];   // [ks & 1][(ks / 2) & 1]; [ct & 1]
  const int tr_row = 8 * h + (l16 >> 2), tr_j = 2 * (g16 & 1) + ((lane & 3) >> 1), tr_in = 8 * (lane & 1);
#pragma unroll
  for (int k = 0; k < 2; k++) {
#pragma unroll
    for (int i = 0; i < 2; i++) p1[k][i] = lane_base(ln, 2 * k + h, i);
    p2lo[k] = lane_base(tr_row, tr_j, k) + tr_in;
    p2hi[k] = lane_base(tr_row + 4, tr_j, k) + tr_in;
  }
  f32x16 acc[C::CT];
#pragma unroll
  for (int ct = 0; ct < C::CT; ct++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[ct][r] = 0.f;

  // ---- a step: the partial scores of tile u meet while phase 1 of tile u + 1 runs, the coefficients of tile u are published,
  // phase 2 of tile u.  What only needs the tile itself is read ahead of the barriers.
  constexpr int PER = C::NI + (STR_STATS ? 1 : 0);   // loads of a tile
  bf16x8 afr[C::KS], bfr[C::CT][2];
  f32x16 s;
  auto load_a = [&](unsigned so) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < C::KS; ks++) afr[ks] = *(const bf16x8*)(smem + p1[ks & 1][(ks >> 1) & 1] + so + 64 * (ks >> 1));
  };
  // this wave's part of S^T[32 streamed x 32 owner]; register 4 j + i of lane (ln, h): streamed row 8 j + 4 h + i
  auto phase1 = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < C::KS; ks++) s = mfma32(afr[ks], ofrag[ks], s);
  };
  f32x4 own = {0.f, 0.f, 0.f, 0.f};
  auto publish_s = [&]() __attribute__((always_inline)) {   // wave j finishes registers 4 j .. 4 j + 3
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const f32x4 v = {s[4 * j], s[4 * j + 1], s[4 * j + 2], s[4 * j + 3]};
      if (j == w) own = v;
      else *(f32x4*)(smem + C::X_OFF + j * 3072 + ((w ^ j) - 1) * 1024 + lane * 16) = v;
    }
  };
  if (nt > 2) wait_vmem<2 * PER>();
  else if (nt > 1) wait_vmem<PER>();
  else wait_vmem<0>();
  load_a(0);
  phase1();
  publish_s();
  int stage = 0;
#pragma unroll 1
  for (int u = 0; u < nt; u++) {
    const int stage1 = stage + 1 == GF_STAGES ? 0 : stage + 1;
    const unsigned so = stage * C::STAGE;
    if (u + 2 < nt) wait_vmem<PER>();   // tile u + 1 has landed
    else wait_vmem<0>();
#pragma unroll
    for (int ct = 0; ct < C::CT; ct++)
#pragma unroll
      for (int kk = 0; kk < 2; kk++) {
        const unsigned off = so + 64 * ct + kk * 16 * C::LDB;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(smem + p2lo[ct & 1] + off));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(smem + p2hi[ct & 1] + off));
        const s16x8 b = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        bfr[ct][kk] = __builtin_bit_cast(bf16x8, b);
      }
    const int t0 = sbeg + u * GF_T, b0 = t0 + 8 * w + 4 * h;   // first of this lane's 4 streamed rows
    f32x4 lse_r = {0.f, 0.f, 0.f, 0.f}, g;
    i32x4 pos_r = {-1, -1, -1, -1};
    if (MERGE && !OWNER_IS_Q) {
      lse_r = *(const f32x4*)(lds_lse + u * GF_T + 8 * w + 4 * h);
      pos_r = *(const i32x4*)(lds_pos + u * GF_T + 8 * w + 4 * h);
    } else if (STR_STATS) {
      const unsigned char* st = smem + w * GF_STAGES * C::STAGE + so + 16 * h;
      lse_r = *(const f32x4*)st;
      if (!OWNER_IS_Q) pos_r = *(const i32x4*)(st + 32);
    }
    load_a(stage1 * C::STAGE);   // (behind the last tile: whatever the stage holds, and nothing uses the scores)
    __syncthreads();
    f32x4 x[3];
#pragma unroll
    for (int k = 0; k < 3; k++) x[k] = *(const f32x4*)(smem + C::X_OFF + (w * 3 + k) * 1024 + lane * 16);
    phase1();
    const f32x4 sv = ((own + x[0]) + x[1]) + x[2];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float t = sv[e] * ga.alpha2;
      if constexpr (SYM) g[e] = one_exp ? fast_exp2(t) * (lse_a + lse_r[e]) : fast_exp2(t - (lse_a + 1.f)) + fast_exp2(t - (lse_r[e] + 1.f));
      else g[e] = fast_exp2(t - (OWNER_IS_Q ? lse_a : lse_r[e]));
      // 0 at the positive (its term is added in fp32 by the kernel that sums the partials, see PosFix), past the end of the
      // split and on the diagonal
      const bool hit = OWNER_IS_Q ? r_a == b0 + e : pos_r[e] == a_q;
      if (hit || b0 + e >= send || (ga.mask_self && b0 + e == a_q)) g[e] = 0.f;
    }
    // A fragments of phase 2 (k = streamed rows): this lane's four are elements 4 h .. of lane 32 (w & 1) + ln, k-step w / 2
    *(bf16x4*)(smem + C::G_OFF + (w >> 1) * 1024 + (32 * (w & 1) + ln) * 16 + 8 * h) = __builtin_convertvector(g, bf16x4);
    __syncthreads();
    publish_s();   // (everybody has read the partial scores of tile u)
    bf16x8 gf[2];
#pragma unroll
    for (int kk = 0; kk < 2; kk++) gf[kk] = *(const bf16x8*)(smem + C::G_OFF + kk * 1024 + lane * 16);
    if (u + GF_STAGES < nt) prefetch(u + GF_STAGES, stage);   // (the stage is this wave's alone, and has been read)
#pragma unroll
    for (int ct = 0; ct < C::CT; ct++)
#pragma unroll
      for (int kk = 0; kk < 2; kk++) acc[ct] = mfma32(gf[kk], bfr[ct][kk], acc[ct]);
    stage = stage1;
  }

  float* out = OWNER_IS_Q ? (ga.dq_out + (size_t)split * ga.dq_split_stride) : (ga.dp_out + (size_t)split * ga.dp_split_stride);
  // (owner rows on M: a register of the wave is two whole 128-byte lines.  With the rows in lanes, 16-byte stores of 32-byte pieces:
  // 13.3 us at 128 x 256 x 768, 12.0 so.)
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const int a = a0 + 8 * (r >> 2) + 4 * h + (r & 3);
    if (a < No) {
#pragma unroll
      for (int ct = 0; ct < C::CT; ct++) out[(size_t)a * D + w * C::DS + 32 * ct + ln] = acc[ct][r] * ga.out_scale;
    }
  }
  chk.finish(ga);
}

// Workgroup `o` of `n` -> task, such that an XCD (ids go to the eight round-robin) has a contiguous range.
__device__ __forceinline__ int xcd_share(int o, int n) {
  const int x = o % 8, more = n % 8;
  return x * (n / 8) + (x < more ? x : more) + o / 8;
}
// A grid of one round is numbered through both roles: an XCD then fetches the code of one of them (with a share of either 32 x 2048
// x 768 takes 27.6 us for 25.3, the 180 shapes of one round 1 % more).  Beyond a round every XCD gets its share of
// either, those with the longer walks first: otherwise the long walks are all on one or two XCDs, two rounds of them there
// (128 x 8192 x 768, 64 walks of 512 rows and 256 of 128: 84.7 us a call, 60.1 so; 8192 x 128 x 768 125.5 and 98.0).
__device__ __forceinline__ int few_spread_id(const GradArgs& ga) {
  const int nQ = ga.obQ * ga.nsq, nP = ga.obP * ga.nsp, id = (int)blockIdx.x;
  if (ga.p_stream_len > ga.q_stream_len) return id < nP ? nQ + xcd_share(id, nP) : xcd_share(id - nP, nQ);
  return id < nQ ? xcd_share(id, nQ) : nQ + xcd_share(id - nQ, nP);
}
template <int D, bool SYM, bool MERGE>
__global__ void __launch_bounds__(256) grad_few_kernel(GradArgs ga, FewMerge fm) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gsmem[];
  const int nQ = ga.obQ * ga.nsq;
  constexpr unsigned ROUND = (D <= 256 ? 2 : 1) * kNumCUDefault;   // workgroups that run at once, by their LDS
  int id = xcd_task_id();
  if (__builtin_expect(gridDim.x > ROUND, 0)) id = few_spread_id(ga);
  if (id < nQ) {
    grad_few_body<D, true, SYM, MERGE>(ga, fm, id % ga.obQ, id / ga.obQ, gsmem);
  } else {
    const int t = id - nQ;
    grad_few_body<D, false, SYM, MERGE>(ga, fm, t % ga.obP, t / ga.obP, gsmem);
  }
}
template <int D, bool SYM, bool MERGE>
static hipError_t grad_few_as(const GradArgs& ga, const FewMerge& fm, int nwg, hipStream_t stream) {
  constexpr int smem = FewCfg<D, MERGE>::SMEM;
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)grad_few_kernel<D, SYM, MERGE>, smem, attr_done); e != hipSuccess) return e;
  grad_few_kernel<D, SYM, MERGE><<<nwg, 256, smem, stream>>>(ga, fm);
  return hipGetLastError();
}
template <int D>
static hipError_t grad_few_of(const GradArgs& ga, const FewMerge& fm, int nwg, hipStream_t stream) {
  if (ga.lse2_t) return grad_few_as<D, true, false>(ga, fm, nwg, stream);
  return fm.splits ? grad_few_as<D, false, true>(ga, fm, nwg, stream) : grad_few_as<D, false, false>(ga, fm, nwg, stream);
}
hipError_t grad_few_launch(const GradArgs& ga, const FewMerge& fm, int d, int nwg, hipStream_t stream) {
  switch (d) {
    case 128: return grad_few_of<128>(ga, fm, nwg, stream);
    case 256: return grad_few_of<256>(ga, fm, nwg, stream);
    case 384: return grad_few_of<384>(ga, fm, nwg, stream);
    case 512: return grad_few_of<512>(ga, fm, nwg, stream);
    case 640: return grad_few_of<640>(ga, fm, nwg, stream);
    case 768: return grad_few_of<768>(ga, fm, nwg, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gc
