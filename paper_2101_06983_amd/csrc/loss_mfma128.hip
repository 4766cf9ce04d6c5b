// bf16 MFMA kernels of the loss path for d = 128 (gfx950): gradient pass and statistics pass.
#include "mfma_common.h"
#include "stats_tile.h"

namespace gc {

// ===========================================================================
// Gradient pass for d = 128 (the NT-Xent workload).  At this width a wave holds whole owner rows, so nothing is exchanged
// between waves: a workgroup (4 waves) owns 128 rows, each wave 32 of them with all 128 columns in registers (MFMA B
// fragments), and the four share the streamed tiles (64 rows, 16 KB) through an LDS ring of four stages.  Per 32 streamed
// rows and wave:
//   phase 1  S^T[32 streamed x 32 owner] = R_tile * O^T, 8 MFMAs 32x32x16.  Lane (n, h) then holds, for owner row n, the
//            scores of streamed rows 8 j + 4 h + i (j, i = 0..3): registers 8 kk .. 8 kk + 7 are streamed rows
//            16 kk + {4 h .. 4 h + 3, 8 + 4 h .. 8 + 4 h + 3}.
//   g        = the coefficient in place, rounded to bf16: registers 8 kk .. 8 kk + 7 ARE the B fragment
//            (k = those streamed rows, n = owner) of
//   phase 2  dO^T[128 x 32 owner] += R_tile^T * g^T, 8 MFMAs 32x32x16, whose A fragments (columns of the tile, the same
//            streamed rows in the same k order) come from two transposing LDS reads each.
// The contraction order over the streamed rows is thus a permutation that both operands of phase 2 share.
// At most 256 registers a lane, so two workgroups share a CU and one wave's arithmetic runs beside the other's MFMAs.
// Per 32 x 32 scores a wave needs 528 cycles of MFMA, 400 of vector arithmetic (one exponential a score), 16 KB of LDS reads
// (128 cycles of the CU's pipe).  16384 views, one walk with one exponential: 138 us, 137 GFLOP = 1.0 PFLOP/s, matrix pipe 49 %
// and vector issue 43 % busy (64 rows a wave, one wave of 512 registers per SIMD: 216, and 233 with two exponentials).  The order
// of MFMAs and arithmetic, wave priorities and scheduling fences move that by less than 1 %.
// ===========================================================================
constexpr int G1_W = 32, G1_T = 64, G1_STAGES = 4;
constexpr int G1_STAT = 512;                      // a stage starts with lse2[64], then pos_idx[64] of the streamed rows
constexpr int G1_STAGE = G1_STAT + G1_T * 256;    // bytes
constexpr int G1_SMEM = G1_STAGES * G1_STAGE;
// chunk c (16 bytes) of tile row r is stored at chunk position c ^ swz128(r): the low row bits pick the 64-byte quarter, the
// next two the chunk inside it.  Free of bank conflicts for the fragment reads and for the transposing ones.
__device__ __forceinline__ int swz128(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

// the first LANES (16 or 32) lanes of the wave load 16 bytes each to lds_base + lane * 16 (EXEC narrowed inside)
template <int LANES>
__device__ __forceinline__ void dma_lanes(const void* gbase, unsigned voff, unsigned lds_base) {
  unsigned long long keep;
  asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %4\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
               : "=&s"(keep) : "s"(lds_base), "v"(voff), "s"(gbase), "s"((1ull << LANES) - 1) : "memory", "m0");
}

// G1_PLAIN: one direction; G1_SYM: the symmetric forms; G1_SYM1: the same with one exponential a score (see kWideLse)
enum G1Mode { G1_PLAIN, G1_SYM, G1_SYM1 };
template <bool OWNER_IS_Q, G1Mode MODE>
__device__ __forceinline__ void grad128_body(const GradArgs& ga, int oblk, int split, unsigned char* smem) {
  constexpr int D = 128;
  constexpr bool SYM = MODE != G1_PLAIN;
  constexpr bool STR_STATS = SYM || !OWNER_IS_Q;   // as in grad_body
  const float* stat_q = MODE == G1_SYM1 ? ga.wexp : ga.lse2;
  const float* stat_p = MODE == G1_SYM1 ? ga.wexp_t : ga.lse2_t;
  const float* lse_own = (SYM && !OWNER_IS_Q) ? stat_p : stat_q;
  const float* lse_str = (SYM && OWNER_IS_Q) ? stat_p : stat_q;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5, ln = lane & 31;
  const int l16 = lane & 15, g16 = lane >> 4;
  const unsigned short* O = OWNER_IS_Q ? ga.Q : ga.P;
  const unsigned short* R = OWNER_IS_Q ? ga.P : ga.Q;
  const int No = OWNER_IS_Q ? ga.B : ga.Pn, Nr = OWNER_IS_Q ? ga.Pn : ga.B;
  const int slen = OWNER_IS_Q ? ga.q_stream_len : ga.p_stream_len;
  const int a0 = oblk * G1_OWN + w * G1_W;   // this wave's first owner row
  const int sbeg = split * slen, send = min(Nr, sbeg + slen);
  const int nt = (send - sbeg + G1_T - 1) / G1_T;   // >= 1
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)smem);
  const int wu = __builtin_amdgcn_readfirstlane(w);   // the wave index as a scalar

  // ---- loads of a streamed tile: 16 instructions of 4 rows, four per wave; lane -> (row, chunk position) ------
  auto src_of = [&](int k, int max_row) __attribute__((always_inline)) -> unsigned {
    const int row = 16 * w + 4 * k + (lane >> 4);
    return (unsigned)(min(row, max_row) * (D * 2) + ((lane & 15) ^ swz128(row)) * 16);
  };
  unsigned voff[4];   // full tile, with the instruction offset 1024 k pre-subtracted
#pragma unroll
  for (int k = 0; k < 4; k++) voff[k] = src_of(k, G1_T - 1) - 1024u * k;
  // row statistics: lanes 0-15 load lse_str[t0 ..], lanes 16-31 (dP role) pos_pad.  (Up to 32 entries behind the padded
  // arrays are read where a range does not start at a multiple of 64: workspace memory, of rows that are masked.)
  const unsigned stat_off = ((lane & 16) && !OWNER_IS_Q ? (unsigned)((const char*)ga.pos_pad - (const char*)lse_str) : 0u) + 16u * (lane & 15);
  const bool stat_wave = STR_STATS && wu == 0;
  auto prefetch = [&](int u) __attribute__((always_inline)) {   // tile u -> stage u % 4
    const int t0 = sbeg + u * G1_T;
    const unsigned st = lds0 + (u & (G1_STAGES - 1)) * G1_STAGE;
    const unsigned short* tile = R + (size_t)t0 * D;
    if (stat_wave) dma_lanes<OWNER_IS_Q ? 16 : 32>(lse_str + t0, stat_off, st);
    if (t0 + G1_T <= Nr) {
      dma_group<4>(tile, voff, st + G1_STAT + 4096 * wu);
    } else {  // ragged last tile: rows past the end re-read the last valid row (their g is forced to 0)
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const unsigned off = src_of(k, Nr - 1 - t0);
        dma_group<1>(tile, &off, st + G1_STAT + 4096 * wu + 1024 * k);
      }
    }
  };

  // owner rows as phase-1 B fragments: lane (ln, h) holds owner row ln, columns 16 ks + 8 h .. + 7
  bf16x8 ofrag[8];
  const int own_idx = a0 + ln;
  float lse_o = MODE == G1_SYM1 ? 0.f : INFINITY;   // (a row past the end is not stored)
  int r_o = -1;
  {
    const int row = min(own_idx, No - 1);
#pragma unroll
    for (int ks = 0; ks < 8; ks++) ofrag[ks] = *(const bf16x8*)(O + (size_t)row * D + 16 * ks + 8 * h);
    if ((OWNER_IS_Q || SYM) && own_idx < No) lse_o = lse_own[own_idx];
    if (OWNER_IS_Q && own_idx < No) r_o = ga.pos_pad[own_idx];
  }
  // The compiler's own loads end here: it does not see the direct-to-LDS loads below, and a wait of its own for
  // these registers inside the loop would also wait for those.  An empty statement that "uses" every loaded register.
#pragma unroll
  for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(ofrag[ks]));
  asm volatile("" : "+v"(lse_o), "+v"(r_o));

  // per-lane LDS offsets inside a stage's tile; everything else of an address is a compile-time constant
  unsigned pa[8], ta[4][2];
#pragma unroll
  for (int k = 0; k < 8; k++) pa[k] = (unsigned)(ln * 256 + (((2 * k + h) ^ swz128(ln)) * 16));
  // transposing reads: rows 16 kk + 8 e + 4 h + l16 / 4, chunk 4 mt + 2 (g16 & 1) + (l16 & 3) / 2, half l16 & 1
  const int tr_r = 4 * h + (l16 >> 2), tr_c = 2 * (g16 & 1) + ((l16 & 3) >> 1);
#pragma unroll
  for (int mt = 0; mt < 4; mt++)
#pragma unroll
    for (int e = 0; e < 2; e++) ta[mt][e] = (unsigned)((8 * e + tr_r) * 256 + ((4 * mt + tr_c) ^ swz128(8 * e + tr_r)) * 16 + 8 * (l16 & 1));

  f32x16 acc[4];
#pragma unroll
  for (int mt = 0; mt < 4; mt++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[mt][r] = 0.f;

#pragma unroll 1
  for (int u = 0; u < min(nt, G1_STAGES - 1); u++) prefetch(u);

  // ---- software pipeline over 32-row halves of the tiles: half s runs, MFMA by MFMA, phase 1 of half s + 1 beside the
  // arithmetic of half s, then phase 2 of half s.  The fragments of the next MFMAs are read four MFMAs ahead.
  f32x16 sacc[2];     // [half parity]
  bf16x8 pfr[4];      // phase-1 A fragments k, k + 4
  bf16x8 afr[4];      // phase-2 A fragments
  constexpr unsigned TILE = G1_STAT;
  auto load_p = [&](auto k_tag, auto off_tag) __attribute__((always_inline)) {
    constexpr int k = decltype(k_tag)::value;
    pfr[k & 3] = *(const bf16x8*)(smem + pa[k] + decltype(off_tag)::value);
  };
  auto load_a = [&](auto i_tag, auto off_tag) __attribute__((always_inline)) {   // fragment i = 2 mt + kk
    constexpr int i = decltype(i_tag)::value, mt = i / 2, kk = i % 2;
    s16x4 q[2];
#pragma unroll
    for (int e = 0; e < 2; e++) q[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(smem + ta[mt][e] + (decltype(off_tag)::value + kk * 4096)));
    const s16x8 t = {q[0][0], q[0][1], q[0][2], q[0][3], q[1][0], q[1][1], q[1][2], q[1][3]};
    afr[i & 3] = __builtin_bit_cast(bf16x8, t);
  };
  auto half = [&](int u, auto stg_tag, auto half_tag) __attribute__((always_inline)) {
    constexpr int STG = decltype(stg_tag)::value, H = decltype(half_tag)::value, CUR = H, NXT = H ^ 1;
    // stage offsets of this half's rows, of the next half's (phase 1) and of the one after it (its first fragments)
    constexpr unsigned O0 = STG * G1_STAGE + TILE + H * 8192;
    constexpr unsigned O1 = H == 0 ? STG * G1_STAGE + TILE + 8192 : ((STG + 1) & 3) * G1_STAGE + TILE;
    constexpr unsigned O2 = ((STG + 1) & 3) * G1_STAGE + TILE + H * 8192;
    constexpr std::integral_constant<unsigned, O0> o0{};
    constexpr std::integral_constant<unsigned, O1> o1{};
    constexpr std::integral_constant<unsigned, O2> o2{};
    const int t0 = sbeg + u * G1_T + H * 32;   // first streamed row of this half
    f32x4 lse_r[4];
    int pos_ln = -1;
    if (STR_STATS) {
#pragma unroll
      for (int j = 0; j < 4; j++) lse_r[j] = *(const f32x4*)(smem + STG * G1_STAGE + H * 128 + (8 * j + 4 * h) * 4);
      if (!OWNER_IS_Q) pos_ln = *(const int*)(smem + STG * G1_STAGE + 256 + H * 128 + 4 * ln);
    }
    static_for<8>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value;
      if constexpr (i == 0) {
        f32x16 z;
#pragma unroll
        for (int r = 0; r < 16; r++) z[r] = 0.f;
        sacc[NXT] = mfma32(pfr[0], ofrag[0], z);
      } else {
        sacc[NXT] = mfma32(pfr[i & 3], ofrag[i], sacc[NXT]);
      }
#pragma unroll
      for (int x = 2 * i; x < 2 * i + 2; x++) {
        float e;
        if constexpr (MODE == G1_SYM1) {
          e = fast_exp2(sacc[CUR][x] * ga.alpha2) * (lse_o + lse_r[x >> 2][x & 3]);
        } else if constexpr (MODE == G1_SYM) {  // mean of the row softmax and the column softmax
          const float t = sacc[CUR][x] * ga.alpha2;
          e = 0.5f * fast_exp2(t - lse_o) + 0.5f * fast_exp2(t - lse_r[x >> 2][x & 3]);
        } else {
          e = fast_exp2(sacc[CUR][x] * ga.alpha2 - (OWNER_IS_Q ? lse_o : lse_r[x >> 2][x & 3]));
        }
        // an empty statement that "uses" the value keeps the arithmetic inside this round
        asm volatile("" : "+v"(e));
        sacc[CUR][x] = e;
      }
      if constexpr (i < 4) load_p(std::integral_constant<int, i + 4>{}, o1);
      else load_a(std::integral_constant<int, i - 4>{}, o0);
      __builtin_amdgcn_sched_barrier(0);  // the rounds stay in order
    });
    // 0 at the positive (j == r_i: its term is added in fp32 by the kernel that sums the partials, see PosFix), zeros for
    // rows past the end of the split and on the diagonal: few tiles
    bool rare = (t0 + 32 > send) || (ga.mask_self && (t0 < a0 + G1_W) && (t0 + 32 > a0));
    rare = rare || (OWNER_IS_Q ? (unsigned)(r_o - t0) < 32u : (unsigned)(pos_ln - a0) < (unsigned)G1_W);
    if (__builtin_amdgcn_ballot_w64(rare) != 0) {
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int in = 8 * (r >> 2) + 4 * h + (r & 3), m = t0 + in;   // streamed row of this register
        const bool hit = OWNER_IS_Q ? r_o == m : __shfl(pos_ln, in) == own_idx;
        if (hit || m >= send || (ga.mask_self && m == own_idx)) sacc[CUR][r] = 0.f;
      }
    }
    bf16x8 gfr[2];
#pragma unroll
    for (int kk = 0; kk < 2; kk++) {
      typedef __attribute__((ext_vector_type(8))) float f32x8;
      const f32x16& g = sacc[CUR];
      const f32x8 v = {g[8 * kk], g[8 * kk + 1], g[8 * kk + 2], g[8 * kk + 3], g[8 * kk + 4], g[8 * kk + 5], g[8 * kk + 6], g[8 * kk + 7]};
      gfr[kk] = __builtin_convertvector(v, bf16x8);
    }
    static_for<8>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value;
      acc[i / 2] = mfma32(afr[i & 3], gfr[i % 2], acc[i / 2]);
      if constexpr (i < 4) load_a(std::integral_constant<int, i + 4>{}, o0);
      else load_p(std::integral_constant<int, i - 4>{}, o2);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // my loads of tile v have landed; `later` tiles behind it have been started
  auto wait_tile = [&](bool later) __attribute__((always_inline)) {
    if (!later) wait_vmem<0>();
    else if (stat_wave) wait_vmem<5>();
    else wait_vmem<4>();
  };
  {   // phase 1 of the first half
    if (nt > 2) { if (stat_wave) wait_vmem<10>(); else wait_vmem<8>(); }
    else wait_tile(nt > 1);
    __syncthreads();
    constexpr std::integral_constant<unsigned, TILE> first{};
    static_for<4>([&](auto k_tag) __attribute__((always_inline)) { load_p(k_tag, first); });
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; r++) z[r] = 0.f;
    sacc[0] = z;
    static_for<8>([&](auto k_tag) __attribute__((always_inline)) {
      constexpr int k = decltype(k_tag)::value;
      sacc[0] = mfma32(pfr[k & 3], ofrag[k], sacc[0]);
      if constexpr (k < 4) load_p(std::integral_constant<int, k + 4>{}, first);
    });
    constexpr std::integral_constant<unsigned, TILE + 8192> second{};
    static_for<4>([&](auto k_tag) __attribute__((always_inline)) { load_p(k_tag, second); });
  }
  // Iteration u: tile u + 1 is needed (phase 1 of its first half), tile u + 2 may be in flight, tile u + 3 is started into the
  // stage of tile u - 1, which everybody has left at the barrier.  (Behind the last tile the pipeline reads a stage that
  // nobody fills any more and uses nothing of it.)
  auto tile = [&](int u, auto stg_tag) __attribute__((always_inline)) {
    wait_tile(u + 2 < nt);
    __syncthreads();
    if (u + 3 < nt) prefetch(u + 3);
    half(u, stg_tag, std::integral_constant<int, 0>{});
    half(u, stg_tag, std::integral_constant<int, 1>{});
  };
#pragma unroll 1
  for (int u = 0; u < nt; u += 4) {
    tile(u, std::integral_constant<int, 0>{});
    if (u + 1 < nt) tile(u + 1, std::integral_constant<int, 1>{});
    if (u + 2 < nt) tile(u + 2, std::integral_constant<int, 2>{});
    if (u + 3 < nt) tile(u + 3, std::integral_constant<int, 3>{});
  }

  // ---- epilogue: lane (ln, h) holds owner row ln, columns 32 mt + 8 (r / 4) + 4 h + r % 4 -----------------
  float* out = OWNER_IS_Q ? (ga.dq_out + (size_t)split * ga.dq_split_stride) : (ga.dp_out + (size_t)split * ga.dp_split_stride);
  if (own_idx < No) {
#pragma unroll
    for (int mt = 0; mt < 4; mt++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const f32x4 v = {acc[mt][4 * j] * ga.out_scale, acc[mt][4 * j + 1] * ga.out_scale,
                         acc[mt][4 * j + 2] * ga.out_scale, acc[mt][4 * j + 3] * ga.out_scale};
        *(f32x4*)(out + (size_t)own_idx * D + 32 * mt + 8 * j + 4 * h) = v;
      }
  }
}

// ONE_WALK (with SYM): the dQ role alone
template <bool SYM, bool ONE_WALK>
__global__ void __launch_bounds__(256, 2) grad128_kernel(GradArgs ga) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gsmem[];
  check_shared_positives(ga);
  const int nQ = ga.obQ * ga.nsq;
  const int id = xcd_task_id();
  const bool own_q = ONE_WALK || id < nQ;
  const int t = own_q ? id : id - nQ;
  if constexpr (SYM) {
    const bool one_exp = __builtin_amdgcn_readfirstlane(*ga.wide) == 0;   // see kWideLse
    if (own_q && one_exp) grad128_body<true, G1_SYM1>(ga, t % ga.obQ, t / ga.obQ, gsmem);
    else if (own_q) grad128_body<true, G1_SYM>(ga, t % ga.obQ, t / ga.obQ, gsmem);
    else if (!ONE_WALK && one_exp) grad128_body<false, G1_SYM1>(ga, t % ga.obP, t / ga.obP, gsmem);
    else if (!ONE_WALK) grad128_body<false, G1_SYM>(ga, t % ga.obP, t / ga.obP, gsmem);
  } else {
    if (own_q) grad128_body<true, G1_PLAIN>(ga, t % ga.obQ, t / ga.obQ, gsmem);
    else grad128_body<false, G1_PLAIN>(ga, t % ga.obP, t / ga.obP, gsmem);
  }
}

// ===========================================================================
// Statistics pass for d = 128 (Eq. 4's normaliser, the positive's logit and the arg-max, per anchor and split).
// The layout of the d = 128 gradient pass without its second contraction: a workgroup (4 waves) owns 256 anchors,
// each wave 64 of them with all 128 columns in registers, and all four share the streamed target tiles (32 rows)
// through an LDS ring of eight stages.  Lane (n, h) holds, for its two anchors 32 i + n, the scores of 16 of a tile's 32
// targets; the other 16 are in lane (n, h ^ 1).  The running (max, sum, arg-max) of an anchor therefore lives in
// a lane of its own and no lane talks to another before the end of the stream: 16 MFMAs against about 5 vector
// operations per score, which a second workgroup on the same CU runs behind the first one's MFMAs.
// ===========================================================================
constexpr int S1_OWN = 256, S1_OWN_W = 64, S1_T = 32, S1_STAGES = 8;
constexpr int S1_STAGE = S1_T * 256, S1_SMEM = S1_STAGES * S1_STAGE;   // bytes
constexpr int S1_AHEAD = 6;   // tile u is read, tiles u+1 .. u+5 are in flight, tile u+6 goes where tile u-2 was
template <bool ARGMAX>
__global__ void __launch_bounds__(256, 2) stats128_kernel(const unsigned short* __restrict__ Q,
                                                          const unsigned short* __restrict__ Pm,
                                                          const int32_t* __restrict__ pos_idx, int B, int P,
                                                          float alpha2, int mask_self, int n_ablk, int cols_per_split,
                                                          float* __restrict__ part_m, float* __restrict__ part_l,
                                                          int* __restrict__ part_idx, float* __restrict__ pos_t) {
  extern __shared__ __attribute__((aligned(16))) unsigned char s1mem[];
  constexpr int D = 128;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5, ln = lane & 31;
  const int task = xcd_task_id();
  const int ablk = task % n_ablk, split = task / n_ablk;
  const int a0 = ablk * S1_OWN + w * S1_OWN_W;   // this wave's first anchor
  const int sbeg = split * cols_per_split, send = min(P, sbeg + cols_per_split);
  const int nt = (send - sbeg + S1_T - 1) / S1_T;   // >= 1
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)s1mem);
  const int wu = __builtin_amdgcn_readfirstlane(w);

  // anchors as B fragments: lane (ln, h) holds anchor 32 n + ln, columns 16 ks + 8 h .. + 7
  bf16x8 ofrag[2][8];
  int own_idx[2], r_o[2];
#pragma unroll
  for (int n = 0; n < 2; n++) {
    own_idx[n] = a0 + 32 * n + ln;
    const int row = min(own_idx[n], B - 1);
#pragma unroll
    for (int ks = 0; ks < 8; ks++) ofrag[n][ks] = *(const bf16x8*)(Q + (size_t)row * D + 16 * ks + 8 * h);
    r_o[n] = (own_idx[n] < B) ? pos_idx[own_idx[n]] : -1;
  }
  // the compiler's own loads end here (it does not see the direct-to-LDS loads counted by wait_vmem below)
#pragma unroll
  for (int n = 0; n < 2; n++) {
#pragma unroll
    for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(ofrag[n][ks]));
    asm volatile("" : "+v"(r_o[n]));
  }

  // loads of a streamed tile: 8 instructions of 4 rows, two per wave; lane -> (row, chunk position)
  auto src_of = [&](int it, int max_row) __attribute__((always_inline)) -> unsigned {
    const int row = 4 * it + (lane >> 4);
    const int c = (lane & 15) ^ swz128(row);
    return (unsigned)(min(row, max_row) * (D * 2) + c * 16);
  };
  const unsigned voff_full[2] = {src_of(2 * w, S1_T - 1), src_of(2 * w + 1, S1_T - 1)};
  auto prefetch = [&](int u) __attribute__((always_inline)) {
    const int t0 = sbeg + u * S1_T;
    const unsigned st = lds0 + (u & (S1_STAGES - 1)) * S1_STAGE;
    const unsigned short* tile = Pm + (size_t)t0 * D;
    if (t0 + S1_T <= P) {
      dma_group<1>(tile, &voff_full[0], st + (2 * wu) * 1024);
      dma_group<1>(tile, &voff_full[1], st + (2 * wu + 1) * 1024);
    } else {  // ragged last tile: rows past the end re-read the last valid row (masked below)
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const unsigned off = src_of(2 * w + k, P - 1 - t0);
        dma_group<1>(tile, &off, st + (2 * wu + k) * 1024);
      }
    }
  };
  const unsigned sw_ln = swz128(ln);

  float rm[2], rl[2], rpos[2];
  int ridx[2];
  bool got[2];
#pragma unroll
  for (int n = 0; n < 2; n++) { rm[n] = -INFINITY; rl[n] = 0.f; rpos[n] = 0.f; ridx[n] = 0x7fffffff; got[n] = false; }

#pragma unroll 1
  for (int u = 0; u < min(nt, S1_AHEAD); u++) prefetch(u);

#pragma unroll 1
  for (int u = 0; u < nt; u++) {
    // my loads of tile u have landed: two instructions per tile, tiles up to u + S1_AHEAD - 1 have been started
    const int later = min(nt - 1, u + S1_AHEAD - 1) - u;
    if (later >= 5) wait_vmem<10>(); else if (later == 4) wait_vmem<8>(); else if (later == 3) wait_vmem<6>();
    else if (later == 2) wait_vmem<4>(); else if (later == 1) wait_vmem<2>(); else wait_vmem<0>();
    __syncthreads();  // ... and everybody's; everybody is past tile u-1, so the stage of tile u-2 is free
    if (u + S1_AHEAD < nt) prefetch(u + S1_AHEAD);
    const unsigned char* st = s1mem + (u & (S1_STAGES - 1)) * S1_STAGE;
    const int t0 = sbeg + u * S1_T;

    bf16x8 pfr[8];
#pragma unroll
    for (int k = 0; k < 8; k++) pfr[k] = *(const bf16x8*)(st + ln * 256 + (((2 * k + h) ^ (int)sw_ln) * 16));
    f32x16 s[2];
#pragma unroll
    for (int n = 0; n < 2; n++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[n][r] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; k++)
#pragma unroll
      for (int n = 0; n < 2; n++) s[n] = mfma32(pfr[k], ofrag[n][k], s[n]);

    // online statistics; s holds raw dot products, the base-2 logit is alpha2 * s (alpha2 > 0: same order).
    // Register r of lane (ln, h) is target t0 + 8 (r / 4) + 4 h + r % 4: increasing in r.
    // the masks that can touch this tile: few tiles, and one scalar branch for the wave (as a per-lane condition the
    // compiler turns the masking into selects that every tile then pays for)
    bool rare = (t0 + S1_T > send) || (mask_self && t0 < a0 + S1_OWN_W && t0 + S1_T > a0);
    rare = rare || (unsigned)(r_o[0] - t0) < (unsigned)S1_T || (unsigned)(r_o[1] - t0) < (unsigned)S1_T;
    if (__builtin_amdgcn_ballot_w64(rare) != 0) {
#pragma unroll
      for (int n = 0; n < 2; n++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int j = t0 + 8 * (r >> 2) + 4 * h + (r & 3);
          const bool self = mask_self && j == own_idx[n];
          const bool masked = j >= send || self;
          // (a positive that the self-mask removes has the logit -inf: its row loss is then +inf)
          if (j == r_o[n] && j < send) { rpos[n] = self ? -INFINITY : s[n][r] * alpha2; got[n] = true; }
          if (masked) s[n][r] = -INFINITY;
        }
    }
#pragma unroll
    for (int n = 0; n < 2; n++) {
      float tmr = -INFINITY; int tc = 0;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const float t = s[n][r];
        if (ARGMAX) {
          const bool le = t <= tmr;   // strict >: the first (smallest) index attaining the maximum
          tmr = le ? tmr : t;
          tc = le ? tc : r;
        } else {
          tmr = fmaxf(tmr, t);
        }
      }
      if (tmr > -INFINITY) {
        const float tm = tmr * alpha2;
        const float mn = fmaxf(rm[n], tm);
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r++) sum += fast_exp2(__builtin_fmaf(s[n][r], alpha2, -mn));
        rl[n] = rl[n] * fast_exp2(rm[n] - mn) + sum;
        if (ARGMAX && tm > rm[n]) ridx[n] = t0 + 8 * (tc >> 2) + 4 * h + (tc & 3);  // later tiles have larger indices
        rm[n] = mn;
      }
    }
  }

  // the positive's score is seen by exactly one lane of one workgroup
#pragma unroll
  for (int n = 0; n < 2; n++)
    if (got[n] && own_idx[n] < B) pos_t[own_idx[n]] = rpos[n];
  // combine the two half-waves (same anchor, the other 16 targets of every tile), then write the split partial
#pragma unroll
  for (int n = 0; n < 2; n++) {
    const float m2 = __shfl_xor(rm[n], 32), l2 = __shfl_xor(rl[n], 32);
    const int i2 = __shfl_xor(ridx[n], 32);
    stat_merge(rm[n], rl[n], ridx[n], m2, l2, i2);
    if (h == 0 && own_idx[n] < B) {
      const size_t o = (size_t)split * B + own_idx[n];
      part_m[o] = rm[n]; part_l[o] = rl[n]; part_idx[o] = ridx[n];
    }
  }
}

// ===========================================================================
// The same for the symmetric forms: the statistics of both sides from one pass over the scores (see kBothMin).
//   TRI (NT-Xent, q = p = z): the scores of the pairs j > i only.  A workgroup owns a block of 256 rows and walks a range
//   of the rows from the block's first one on.  Inside the block every pair is formed twice (the self mask and the
//   positives are there: views 2 k, 2 k + 1 never lie in different blocks) and counts for the lane's row; beyond it each
//   score counts for its row and its column.
//   otherwise (symmetric loss): owners are anchors, streamed rows are targets, each score counts for both.
// Column sums: 32 lanes hold a column's 32 owners, twice; 54 operations per 32 x 64 tile bring them together
// (reduce16_lanes32), the four waves' sums meet in LDS one tile later.  16384 views: 72 us (all scores for the rows alone: 105).
// ===========================================================================
template <bool TRI>
__global__ void __launch_bounds__(256, 2) stats128_both_kernel(StatsArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char s1mem[];
  constexpr int D = 128;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5, ln = lane & 31;
  both_begin(g);
  int task = xcd_task_id(), ablk, split;
  if (TRI) split = tri_task(task, g.Pn, S1_OWN, g.cols_per_split, ablk);
  else { ablk = task % g.n_ablk; split = task / g.n_ablk; }
  const int blk_end = (ablk + 1) * S1_OWN;
  const int a0 = ablk * S1_OWN + w * S1_OWN_W;   // this wave's first owner
  const int sbeg = (TRI ? ablk * S1_OWN : 0) + split * g.cols_per_split, send = min(g.Pn, sbeg + g.cols_per_split);
  const int nt = (send - sbeg + S1_T - 1) / S1_T;   // >= 1
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)s1mem);
  const int wu = __builtin_amdgcn_readfirstlane(w);
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  f32x2* cbuf = (f32x2*)(s1mem + S1_SMEM);   // [tile parity][wave][32 columns] (maximum, sum)

  bf16x8 ofrag[2][8];
  int own_idx[2], r_o[2];
#pragma unroll
  for (int n = 0; n < 2; n++) {
    own_idx[n] = a0 + 32 * n + ln;
    const int row = min(own_idx[n], g.B - 1);
#pragma unroll
    for (int ks = 0; ks < 8; ks++) ofrag[n][ks] = *(const bf16x8*)(g.Q + (size_t)row * D + 16 * ks + 8 * h);
    r_o[n] = own_idx[n] >= g.B ? -1 : TRI ? own_idx[n] ^ 1 : g.pos_idx[own_idx[n]];
  }
  // the compiler's own loads end here (it does not see the direct-to-LDS loads counted by wait_vmem below)
#pragma unroll
  for (int n = 0; n < 2; n++) {
#pragma unroll
    for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(ofrag[n][ks]));
    asm volatile("" : "+v"(r_o[n]));
  }
  auto src_of = [&](int it, int max_row) __attribute__((always_inline)) -> unsigned {
    const int row = 4 * it + (lane >> 4);
    const int c = (lane & 15) ^ swz128(row);
    return (unsigned)(min(row, max_row) * (D * 2) + c * 16);
  };
  const unsigned voff_full[2] = {src_of(2 * w, S1_T - 1), src_of(2 * w + 1, S1_T - 1)};
  auto prefetch = [&](int u) __attribute__((always_inline)) {
    const int t0 = sbeg + u * S1_T;
    const unsigned st = lds0 + (u & (S1_STAGES - 1)) * S1_STAGE;
    const unsigned short* tile = g.P + (size_t)t0 * D;
    if (t0 + S1_T <= g.Pn) {
      dma_group<1>(tile, &voff_full[0], st + (2 * wu) * 1024);
      dma_group<1>(tile, &voff_full[1], st + (2 * wu + 1) * 1024);
    } else {  // ragged last tile: rows past the end re-read the last valid row (masked below)
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const unsigned off = src_of(2 * w + k, g.Pn - 1 - t0);
        dma_group<1>(tile, &off, st + (2 * wu + k) * 1024);
      }
    }
  };
  const unsigned sw_ln = swz128(ln);
  const int col_in = 8 * (reduce16_reg_of(lane) >> 2) + 4 * h + (reduce16_reg_of(lane) & 3);   // the column this lane ends up with

  float lf[2] = {0.f, 0.f};                              // sums with the reference 0
  float rm[2] = {-INFINITY, -INFINITY}, rl[2] = {0.f, 0.f};   // of the tiles that needed one of their own
  float rpos[2] = {0.f, 0.f};
  bool got[2] = {false, false};
  const bool own_edge = a0 + S1_OWN_W > g.B;

  // the four waves' column sums of tile u - 1, in wave order
  auto flush_cols = [&](int u) __attribute__((always_inline)) {
    const int t0 = sbeg + (u - 1) * S1_T;
    if (u < 1 || (TRI && t0 < blk_end) || wu != ((u - 1) & 3)) return;
    float m = -INFINITY, l = 0.f;
    f32x2 x[4];
#pragma unroll
    for (int k = 0; k < 4; k++) { x[k] = cbuf[(((u - 1) & 1) * 4 + k) * 32 + ln]; m = fmaxf(m, x[k][0]); }
    const float ms = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int k = 0; k < 4; k++) l += x[k][1] * fast_exp2(x[k][0] - ms);
    if (h == 0 && t0 + ln < send) {
      const size_t o = (size_t)ablk * g.Pn + t0 + ln;
      g.col_m[o] = m; g.col_l[o] = l;
    }
  };

#pragma unroll 1
  for (int u = 0; u < min(nt, S1_AHEAD); u++) prefetch(u);

#pragma unroll 1
  for (int u = 0; u < nt; u++) {
    const int later = min(nt - 1, u + S1_AHEAD - 1) - u;
    if (later >= 5) wait_vmem<10>(); else if (later == 4) wait_vmem<8>(); else if (later == 3) wait_vmem<6>();
    else if (later == 2) wait_vmem<4>(); else if (later == 1) wait_vmem<2>(); else wait_vmem<0>();
    lds_barrier();  // everybody's part has landed, and the column sums of tile u-1 too; everybody is past tile u-1, so the stage of tile u-2 is free
    if (u + S1_AHEAD < nt) prefetch(u + S1_AHEAD);
    flush_cols(u);
    const unsigned char* st = s1mem + (u & (S1_STAGES - 1)) * S1_STAGE;
    const int t0 = sbeg + u * S1_T;

    bf16x8 pfr[8];
#pragma unroll
    for (int k = 0; k < 8; k++) pfr[k] = *(const bf16x8*)(st + ln * 256 + (((2 * k + h) ^ (int)sw_ln) * 16));
    f32x16 s[2];
#pragma unroll
    for (int n = 0; n < 2; n++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[n][r] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; k++)
#pragma unroll
      for (int n = 0; n < 2; n++) s[n] = mfma32(pfr[k], ofrag[n][k], s[n]);

    // register r of lane (ln, h) is streamed row t0 + 8 (r / 4) + 4 h + r % 4
    const bool has_pos = (unsigned)(r_o[0] - t0) < (unsigned)S1_T || (unsigned)(r_o[1] - t0) < (unsigned)S1_T;
    if (__builtin_amdgcn_ballot_w64(has_pos) != 0) {
#pragma unroll
      for (int n = 0; n < 2; n++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int j = t0 + 8 * (r >> 2) + 4 * h + (r & 3);
          if (j == r_o[n] && j < send) {
            rpos[n] = s[n][r] * g.alpha2; got[n] = true;
            s[n][r] = -INFINITY;   // the positive is no part of the sums (both_merge_kernel adds it)
          }
        }
    }
    const bool cols = !TRI || t0 >= blk_end;
    bool done = false;
    if (cols && !own_edge && t0 + S1_T <= send) {
      float rs[2], v[16];
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const float e0 = fast_exp2(s[0][r] * g.alpha2), e1 = fast_exp2(s[1][r] * g.alpha2);
        rs[0] = r ? rs[0] + e0 : e0;
        rs[1] = r ? rs[1] + e1 : e1;
        v[r] = e0 + e1;
      }
      const float c = reduce16_lanes32<false>(v, lane);
      const bool in = fminf(fminf(rs[0], rs[1]), c) >= kBothMin && fmaxf(fmaxf(rs[0], rs[1]), c) <= kBothMax;
      if (__builtin_amdgcn_ballot_w64(!in) == 0) {
        lf[0] += rs[0]; lf[1] += rs[1];
        if (!(lane & 1)) cbuf[((u & 1) * 4 + wu) * 32 + col_in] = f32x2{0.f, c};
        done = true;
      }
    }
    if (!done) {   // masks, and references of its own for every row and column
#pragma unroll
      for (int n = 0; n < 2; n++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int j = t0 + 8 * (r >> 2) + 4 * h + (r & 3);
          s[n][r] = (j >= send || own_idx[n] >= g.B || (TRI && j == own_idx[n])) ? -INFINITY : s[n][r] * g.alpha2;
        }
#pragma unroll
      for (int n = 0; n < 2; n++) {
        float tm = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; r++) tm = fmaxf(tm, s[n][r]);
        if (tm > -INFINITY) {
          const float mn = fmaxf(rm[n], tm);
          float sum = 0.f;
#pragma unroll
          for (int r = 0; r < 16; r++) sum += fast_exp2(s[n][r] - mn);
          rl[n] = rl[n] * fast_exp2(rm[n] - mn) + sum;
          rm[n] = mn;
        }
      }
      if (cols) {
        float mx[16], v[16];
#pragma unroll
        for (int r = 0; r < 16; r++) mx[r] = fmaxf(s[0][r], s[1][r]);
#pragma unroll
        for (int r = 0; r < 16; r++) {
          float m = max_lanes32(mx[r]);
          m = m == -INFINITY ? 0.f : m;
          v[r] = fast_exp2(s[0][r] - m) + fast_exp2(s[1][r] - m);
        }
        const float cm = reduce16_lanes32<true>(mx, lane), c = reduce16_lanes32<false>(v, lane);
        if (!(lane & 1)) cbuf[((u & 1) * 4 + wu) * 32 + col_in] = f32x2{cm, c};
      }
    }
  }
  __syncthreads();
  flush_cols(nt);

  // the positive's score is seen by exactly one lane of one workgroup
#pragma unroll
  for (int n = 0; n < 2; n++)
    if (got[n] && own_idx[n] < g.B) g.pos_t[own_idx[n]] = rpos[n];
  // the sums of both kinds, then the two half-waves (same row, the other 16 streamed rows of every tile)
#pragma unroll
  for (int n = 0; n < 2; n++) {
    int unused = 0;
    stat_merge(rm[n], rl[n], unused, lf[n] > 0.f ? 0.f : -INFINITY, lf[n], 0);
    const float m2 = __shfl_xor(rm[n], 32), l2 = __shfl_xor(rl[n], 32);
    stat_merge(rm[n], rl[n], unused, m2, l2, 0);
    if (h == 0 && own_idx[n] < g.B) {
      const size_t o = (size_t)split * g.B + own_idx[n];
      g.row_m[o] = rm[n]; g.row_l[o] = rl[n];
    }
  }
}
template <bool TRI>
static hipError_t stats128_both_launch(const StatsArgs& g, int nwg, hipStream_t stream) {
  constexpr int smem = S1_SMEM + 2 * 4 * 32 * 8;
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)stats128_both_kernel<TRI>, smem, attr_done); e != hipSuccess) return e;
  stats128_both_kernel<TRI><<<nwg, 256, smem, stream>>>(g);
  return hipGetLastError();
}
hipError_t launch_stats128_both(const StatsArgs& g, bool triangle, int nwg, hipStream_t stream) {
  return triangle ? stats128_both_launch<true>(g, nwg, stream) : stats128_both_launch<false>(g, nwg, stream);
}

template <bool ARGMAX>
static hipError_t stats128_launch(const LossArgs& a, const LossPlan& pl) {
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)stats128_kernel<ARGMAX>, S1_SMEM, attr_done); e != hipSuccess) return e;
  char* ws = a.ws;
  const int n_ablk = (a.B + S1_OWN - 1) / S1_OWN;
  stats128_kernel<ARGMAX><<<n_ablk * pl.stat_splits, 256, S1_SMEM, a.stream>>>(
      (const unsigned short*)a.q, (const unsigned short*)a.p, a.pos_idx, a.B, a.P, a.alpha * kLog2e,
      (a.flags & GC_MASK_SELF) ? 1 : 0, n_ablk, pl.stat_cols_per_split, (float*)(ws + pl.off_part_m),
      (float*)(ws + pl.off_part_l), (int*)(ws + pl.off_part_idx), (float*)(ws + pl.off_pos));
  return hipGetLastError();
}
hipError_t launch_stats128(const LossArgs& a, const LossPlan& pl) {
  return a.argmax ? stats128_launch<true>(a, pl) : stats128_launch<false>(a, pl);
}

template <bool SYM, bool ONE_WALK>
static hipError_t grad128_launch_as(const GradArgs& ga, int nwg, hipStream_t stream) {
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)grad128_kernel<SYM, ONE_WALK>, G1_SMEM, attr_done); e != hipSuccess) return e;
  grad128_kernel<SYM, ONE_WALK><<<nwg, 256, G1_SMEM, stream>>>(ga);
  return hipGetLastError();
}
hipError_t grad128_launch(const GradArgs& ga, int nwg, hipStream_t stream) {
  if (!ga.lse2_t) return grad128_launch_as<false, false>(ga, nwg, stream);
  return ga.obP ? grad128_launch_as<true, false>(ga, nwg, stream) : grad128_launch_as<true, true>(ga, nwg, stream);
}

}  // namespace gc
