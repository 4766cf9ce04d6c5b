// bf16 MFMA kernels of the loss path for d = 128 (gfx950): gradient pass and statistics pass.
#include "mfma_common.h"
#include "stats_tile.h"

namespace gc {

// ===========================================================================
// Gradient pass for d = 128 (the NT-Xent workload).  At this width a wave can hold whole owner rows, so
// nothing is exchanged between waves: a workgroup (4 waves, one per SIMD) owns 256 rows, each wave 64 of
// them with all 128 columns in registers (64 VGPRs as MFMA B fragments), and all four share the streamed
// tiles (32 rows x 128 columns, 8 KB) through one LDS ring of four stages.  Per tile and wave:
//   phase 1  S^T[32 streamed x 64 owner] = R_tile * O^T, 16 MFMAs 32x32x16.  Lane (n, h) then holds, for owner
//            row n, the scores of streamed rows 8 j + 4 h + i (j, i = 0..3): registers 8 kk .. 8 kk + 7 are
//            streamed rows 16 kk + {4 h .. 4 h + 3, 8 + 4 h .. 8 + 4 h + 3}.
//   g        = 2^(t - lse2) - [j = r_i] in place, rounded to bf16: registers 8 kk .. 8 kk + 7 ARE the B
//            fragment (k = those streamed rows, n = owner) of
//   phase 2  dO^T[128 x 64 owner] += R_tile^T * g^T, 16 MFMAs 32x32x16, whose A fragments (columns of the tile,
//            the same streamed rows in the same k order) come from two transposing LDS reads each.
// The contraction order over the streamed rows is thus a permutation that both operands of phase 2 share.
// LDS per tile: every wave reads the tile twice (8 KB + 8 KB), 72 KB per workgroup against 64 MFMAs per SIMD.
// ===========================================================================
constexpr int G1_OWN_W = 64, G1_T = 32, G1_STAGES = 8, G1_AHEAD = 6;  // tiles u-1 .. u+1 alive, up to u+5 started
constexpr int G1_STAT = 256;                      // a stage starts with lse2[32], then pos_idx[32] of the streamed rows
constexpr int G1_STAGE = G1_STAT + G1_T * 256;    // bytes
constexpr int G1_SMEM = G1_STAGES * G1_STAGE;
// chunk c (16 bytes) of tile row r is stored at chunk position c ^ swz128(r): 8 consecutive rows of a
// fragment read, and the 4 rows x 2 chunks of a transposing read, fall into different 16-byte bank groups.
// (The bank-conflict counter still shows a conflict on every second LDS cycle of these kernels.  4-bit maps that remove
// them all -- e.g. ((row & 3) << 2) | ((row >> 2) & 3): the low row bits pick the 64-byte quarter, the next two the
// chunk inside it -- were measured on the kernels themselves: LDS cycles halved, waits for LDS a tenth, the time of the
// gradient kernel equal within 1 %.  With a 3-bit map fragment k + 4 of a row sits a fixed 128 bytes behind fragment k,
// an immediate offset; a 4-bit map needs a second set of address registers, which this kernel, at 512 of 512, does not
// have: it spills again.  The loop is paced by its barrier and the waits for the tile loads, not by LDS.)
__device__ __forceinline__ int swz128(int row) { return ((row & 3) << 1) | ((row >> 2) & 1); }

// the first `LANES` lanes of the wave load 16 bytes each to lds_base + lane * 16 (EXEC narrowed inside)
__device__ __forceinline__ void dma_lanes16(const void* gbase, unsigned voff, unsigned lds_base) {
  unsigned long long keep;
  asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, 0xffff\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
               : "=&s"(keep) : "s"(lds_base), "v"(voff), "s"(gbase) : "memory", "m0");
}

template <bool OWNER_IS_Q, bool SYM>
__device__ __forceinline__ void grad128_body(const GradArgs& ga, int oblk, int split, unsigned char* smem) {
  constexpr int D = 128;
  constexpr bool STR_STATS = SYM || !OWNER_IS_Q;   // as in grad_body
  const float* lse_own = (SYM && !OWNER_IS_Q) ? ga.lse2_t : ga.lse2;
  const float* lse_str = (SYM && OWNER_IS_Q) ? ga.lse2_t : ga.lse2;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, h = lane >> 5, ln = lane & 31;
  const int l16 = lane & 15, g16 = lane >> 4;
  const unsigned short* O = OWNER_IS_Q ? ga.Q : ga.P;
  const unsigned short* R = OWNER_IS_Q ? ga.P : ga.Q;
  const int No = OWNER_IS_Q ? ga.B : ga.Pn, Nr = OWNER_IS_Q ? ga.Pn : ga.B;
  const int slen = OWNER_IS_Q ? ga.q_stream_len : ga.p_stream_len;
  const int a0 = oblk * G1_OWN + w * G1_OWN_W;   // this wave's first owner row
  const int sbeg = split * slen, send = min(Nr, sbeg + slen);
  const int nt = (send - sbeg + G1_T - 1) / G1_T;   // >= 1
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)smem);
  const int wu = __builtin_amdgcn_readfirstlane(w);   // the wave index as a scalar

  // owner rows as phase-1 B fragments: lane (ln, h) holds owner row 32 n + ln, columns 16 ks + 8 h .. + 7
  bf16x8 ofrag[2][8];
  int own_idx[2];
  float lse_o[2]; int r_o[2];
#pragma unroll
  for (int n = 0; n < 2; n++) {
    own_idx[n] = a0 + 32 * n + ln;
    const int row = min(own_idx[n], No - 1);
#pragma unroll
    for (int ks = 0; ks < 8; ks++) ofrag[n][ks] = *(const bf16x8*)(O + (size_t)row * D + 16 * ks + 8 * h);
    lse_o[n] = INFINITY; r_o[n] = -1;            // a row past the end: g = 0
    if ((OWNER_IS_Q || SYM) && own_idx[n] < No) lse_o[n] = lse_own[own_idx[n]];
    if (OWNER_IS_Q && own_idx[n] < No) r_o[n] = ga.pos_pad[own_idx[n]];
  }
  // The compiler's own loads end here: it does not see the direct-to-LDS loads below, and a wait of its own for
  // these registers inside the loop would also wait for those.  An empty statement that "uses" every loaded register.
#pragma unroll
  for (int n = 0; n < 2; n++) {
#pragma unroll
    for (int ks = 0; ks < 8; ks++) asm volatile("" : "+v"(ofrag[n][ks]));
    asm volatile("" : "+v"(lse_o[n]), "+v"(r_o[n]));
  }

  // ---- loads of a streamed tile: 8 instructions of 4 rows, two per wave; lane -> (row, chunk position) ------
  auto src_of = [&](int it, int max_row) __attribute__((always_inline)) -> unsigned {
    const int row = 4 * it + (lane >> 4);
    const int c = (lane & 15) ^ swz128(row);
    return (unsigned)(min(row, max_row) * (D * 2) + c * 16);
  };
  const unsigned voff_full[2] = {src_of(2 * w, G1_T - 1), src_of(2 * w + 1, G1_T - 1)};
  const unsigned stat_off = ((lane & 8) && !OWNER_IS_Q) ? (unsigned)((const char*)ga.pos_pad - (const char*)ga.lse2) + 16u * (lane & 7) : 16u * (lane & 7);
  const bool stat_wave = STR_STATS && wu == 0;
  auto prefetch = [&](int u) __attribute__((always_inline)) {   // tile u -> stage u % 4
    const int t0 = sbeg + u * G1_T;
    const unsigned st = lds0 + (u & (G1_STAGES - 1)) * G1_STAGE;
    const unsigned short* tile = R + (size_t)t0 * D;
    if (stat_wave) dma_lanes16(lse_str + t0, stat_off, st);
    if (t0 + G1_T <= Nr) {
      dma_group<1>(tile, &voff_full[0], st + G1_STAT + (2 * wu) * 1024);
      dma_group<1>(tile, &voff_full[1], st + G1_STAT + (2 * wu + 1) * 1024);
    } else {  // ragged last tile: rows past the end re-read the last valid row (their g is forced to 0)
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const unsigned off = src_of(2 * w + k, Nr - 1 - t0);
        dma_group<1>(tile, &off, st + G1_STAT + (2 * wu + k) * 1024);
      }
    }
  };

  // per-lane LDS addresses inside a stage
  const unsigned sw_ln = swz128(ln);
  // transposing reads: rows 16 kk + 8 e + 4 h + (l16 >> 2), chunk 4 mt + 2 (g16 & 1) + ((l16 & 3) >> 1), half l16 & 1
  const int tr_r = 4 * h + (l16 >> 2), tr_c = 2 * (g16 & 1) + ((l16 & 3) >> 1);
  unsigned troff[2][2];  // [kk][e]: the swizzle depends on the row, so one base per (kk, e); + 64 * mt
#pragma unroll
  for (int kk = 0; kk < 2; kk++)
#pragma unroll
    for (int e = 0; e < 2; e++) {
      const int row = 16 * kk + 8 * e + tr_r;
      troff[kk][e] = G1_STAT + row * 256 + 8 * (l16 & 1);   // chunk part added per mt (it is swizzled)
    }

  f32x16 acc[4][2];
#pragma unroll
  for (int mt = 0; mt < 4; mt++)
#pragma unroll
    for (int n = 0; n < 2; n++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[mt][n][r] = 0.f;

  // ---- software pipeline over the tiles: iteration u interleaves, MFMA by MFMA, phase 1 of tile u+1, the
  // exp2 arithmetic of tile u (whose scores iteration u-1 left in registers) and phase 2 of tile u-1 (whose g the
  // previous iteration left as fragments): a wave's VALU work hides behind its own MFMAs only when interleaved.
  // Tiles u-1, u, u+1 are alive in the ring, u+2 .. u+5 in flight.
  f32x16 sacc[2][2];     // [tile parity][owner half]
  bf16x8 gfr[2][2];      // g of the tile last through the softmax: [owner half][kk]
#pragma unroll
  for (int n = 0; n < 2; n++)
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int e = 0; e < 8; e++) gfr[n][kk][e] = 0;

#pragma unroll 1
  for (int u = 0; u < min(nt, G1_AHEAD - 1); u++) prefetch(u);   // iteration -1 starts tile G1_AHEAD - 1

  // PT: parity of tile u+1 (where phase 1 writes); the softmax reads parity PT ^ 1
  // STEADY: all three parts are live (1 <= u, u + 1 < nt): no branches inside the MFMA stream
  auto body = [&](int u, auto pt_tag, auto steady_tag) __attribute__((always_inline)) {
    constexpr int PT = decltype(pt_tag)::value;
    constexpr bool STEADY = decltype(steady_tag)::value;
    const bool p1 = STEADY || (u + 1 < nt), sm = STEADY || (u >= 0 && u < nt), p2 = STEADY || (u >= 1);
    // my loads of tile u+1 have landed (tiles up to u + G1_AHEAD - 1 have been started)
    if (p1) {
      const int later = min(nt - 1, u + G1_AHEAD - 1) - (u + 1);   // tiles started after u+1: 0 .. G1_AHEAD - 2
      if (stat_wave) { if (later >= 4) wait_vmem<12>(); else if (later == 3) wait_vmem<9>(); else if (later == 2) wait_vmem<6>(); else if (later == 1) wait_vmem<3>(); else wait_vmem<0>(); }
      else { if (later >= 4) wait_vmem<8>(); else if (later == 3) wait_vmem<6>(); else if (later == 2) wait_vmem<4>(); else if (later == 1) wait_vmem<2>(); else wait_vmem<0>(); }
    }
    __syncthreads();  // ... and everybody's; everybody is done with tile u-2, whose stage is loaded next
    if (u + G1_AHEAD < nt) prefetch(u + G1_AHEAD);
    const unsigned char* st_p1 = smem + ((u + 1) & (G1_STAGES - 1)) * G1_STAGE;
    const unsigned char* st_sm = smem + (u & (G1_STAGES - 1)) * G1_STAGE;
    const unsigned char* st_p2 = smem + ((u - 1) & (G1_STAGES - 1)) * G1_STAGE;
    const int t0 = sbeg + u * G1_T;   // first streamed row of tile u

    // fragments: row statistics of tile u, then tile u+1 for phase 1 and transposed tile u-1 for phase 2 in
    // the order in which the rounds below consume them (LDS returns reads in order, and the 24 reads of the
    // four waves keep the LDS busy for most of an iteration: the first MFMAs must not wait for the last read)
    f32x4 lse_r[4]; i32x4 pos_r[4];
    if (STR_STATS && sm) {
#pragma unroll
      for (int j = 0; j < 4; j++) {
        lse_r[j] = *(const f32x4*)(st_sm + (8 * j + 4 * h) * 4);
        if (!OWNER_IS_Q) pos_r[j] = *(const i32x4*)(st_sm + 128 + (8 * j + 4 * h) * 4);
      }
    }
    bf16x8 pfr[8];
    bf16x8 afr[4][2];
    // round 2 k needs pfr[k] and afr[k / 2][k % 2]: the first four pairs are read here, pair k + 4 behind round 2 k + 1,
    // into the registers that pair k has just left (all eight at once cost 32 registers that the loop does not have)
    auto load_pair = [&](auto k_tag) __attribute__((always_inline)) {
      constexpr int k = decltype(k_tag)::value;
      if (p1) pfr[k] = *(const bf16x8*)(st_p1 + G1_STAT + ln * 256 + (((2 * k + h) ^ (int)sw_ln) * 16));
      if (p2) {
        constexpr int mt = k / 2, kk = k % 2;
        s16x4 q[2];
#pragma unroll
        for (int e = 0; e < 2; e++) {
          const int row = 16 * kk + 8 * e + tr_r;
          const int c = (4 * mt + tr_c) ^ swz128(row);
          q[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(st_p2 + troff[kk][e] + c * 16));
        }
        s16x8 t = {q[0][0], q[0][1], q[0][2], q[0][3], q[1][0], q[1][1], q[1][2], q[1][3]};
        afr[mt][kk] = __builtin_bit_cast(bf16x8, t);
      }
    };
    static_for<4>(load_pair);
    // 16 rounds: one phase-1 MFMA pair position, one phase-2 MFMA, the exp2 of two scores
    static_for<16>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value;
      if (p1) {
        constexpr int ks = i / 2, n = i % 2;
        if constexpr (ks == 0) {
          f32x16 z;
#pragma unroll
          for (int r = 0; r < 16; r++) z[r] = 0.f;
          sacc[PT][n] = mfma32(pfr[ks], ofrag[n][ks], z);
        } else {
          sacc[PT][n] = mfma32(pfr[ks], ofrag[n][ks], sacc[PT][n]);
        }
      }
      if (p2) {
        constexpr int mt = i / 4, kk = (i / 2) % 2, n = i % 2;
        acc[mt][n] = mfma32(afr[mt][kk], gfr[n][kk], acc[mt][n]);
      }
      if (sm) {
#pragma unroll
        for (int n = 0; n < 2; n++) {
          float e;
          if constexpr (SYM) {  // mean of the row softmax and the column softmax (folding the halves into the
            // exponents saves two operations per score and measured slower here: 8 % while the kernel spilled, 1 % since)
            const float t = sacc[PT ^ 1][n][i] * ga.alpha2;
            e = 0.5f * fast_exp2(t - lse_o[n]) + 0.5f * fast_exp2(t - lse_r[i >> 2][i & 3]);
          } else {
            const float l = OWNER_IS_Q ? lse_o[n] : lse_r[i >> 2][i & 3];
            e = fast_exp2(sacc[PT ^ 1][n][i] * ga.alpha2 - l);
          }
          // an empty statement that "uses" the value: it keeps the arithmetic inside this round (pure
          // arithmetic would otherwise be moved behind all the MFMAs and run exposed)
          if constexpr (STEADY) asm volatile("" : "+v"(e));
          sacc[PT ^ 1][n][i] = e;
        }
      }
      if constexpr (i % 2 == 1 && i / 2 + 4 < 8) load_pair(std::integral_constant<int, i / 2 + 4>{});
      if constexpr (STEADY) __builtin_amdgcn_sched_barrier(0);  // the rounds stay in order
    });
    if (sm) {
      // 0 at the positive (j == r_i: its term is added in fp32 by the kernel that sums the partials, see PosFix),
      // zeros for rows past the end of the split and on the diagonal: few tiles
      bool rare = (t0 + G1_T > send) || (ga.mask_self && (t0 < a0 + G1_OWN_W) && (t0 + G1_T > a0));
      if (OWNER_IS_Q) {
        rare = rare || (unsigned)(r_o[0] - t0) < (unsigned)G1_T || (unsigned)(r_o[1] - t0) < (unsigned)G1_T;
      } else {
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
          for (int e = 0; e < 4; e++) rare = rare || (unsigned)(pos_r[j][e] - a0) < (unsigned)G1_OWN_W;
      }
      if (__builtin_amdgcn_ballot_w64(rare) != 0) {
#pragma unroll
        for (int n = 0; n < 2; n++)
#pragma unroll
          for (int r = 0; r < 16; r++) {
            const int m = t0 + 8 * (r >> 2) + 4 * h + (r & 3);   // streamed row of this register
            const bool hit = OWNER_IS_Q ? (r_o[n] == m) : (pos_r[r >> 2][r & 3] == own_idx[n]);
            if (hit || m >= send || (ga.mask_self && m == own_idx[n])) sacc[PT ^ 1][n][r] = 0.f;
          }
      }
    }
    // the phase-2 MFMAs above have read the old fragments: now they take the g of tile u
    if (sm) {
#pragma unroll
      for (int n = 0; n < 2; n++)
#pragma unroll
        for (int kk = 0; kk < 2; kk++) {
          typedef __attribute__((ext_vector_type(8))) float f32x8;
          const f32x16& g = sacc[PT ^ 1][n];
          const f32x8 v = {g[8 * kk], g[8 * kk + 1], g[8 * kk + 2], g[8 * kk + 3], g[8 * kk + 4], g[8 * kk + 5], g[8 * kk + 6], g[8 * kk + 7]};
          gfr[n][kk] = __builtin_convertvector(v, bf16x8);
        }
    }
  };
  // iterations u = -1 .. nt (phase 1 of tile 0 first, phase 2 of tile nt-1 last), two per trip so that the
  // parity of the score registers is a compile-time constant
  constexpr std::integral_constant<int, 0> pt0{};   // u odd: tile u+1 has parity 0
  constexpr std::integral_constant<int, 1> pt1{};
  body(-1, pt0, std::false_type{});
  body(0, pt1, std::false_type{});
  int u = 1;
#pragma unroll 1
  for (; u + 2 < nt; u += 2) {
    body(u, pt0, std::true_type{});
    body(u + 1, pt1, std::true_type{});
  }
#pragma unroll 1
  for (; u <= nt; u += 2) {
    body(u, pt0, std::false_type{});
    if (u + 1 <= nt) body(u + 1, pt1, std::false_type{});
  }

  // ---- epilogue: lane (ln, h) holds owner row 32 n + ln, columns 32 mt + 8 (r / 4) + 4 h + r % 4 -----------------
  float* out = OWNER_IS_Q ? (ga.dq_out + (size_t)split * ga.dq_split_stride) : (ga.dp_out + (size_t)split * ga.dp_split_stride);
#pragma unroll
  for (int n = 0; n < 2; n++) {
    if (own_idx[n] < No) {
#pragma unroll
      for (int mt = 0; mt < 4; mt++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const f32x4 v = {acc[mt][n][4 * j] * ga.out_scale, acc[mt][n][4 * j + 1] * ga.out_scale,
                           acc[mt][n][4 * j + 2] * ga.out_scale, acc[mt][n][4 * j + 3] * ga.out_scale};
          *(f32x4*)(out + (size_t)own_idx[n] * D + 32 * mt + 8 * j + 4 * h) = v;
        }
    }
  }
}

template <bool SYM>
__global__ void __launch_bounds__(256) grad128_kernel(GradArgs ga) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gsmem[];
  check_shared_positives(ga);
  const int nQ = ga.obQ * ga.nsq;
  const int id = xcd_task_id();
  if (id < nQ) {
    grad128_body<true, SYM>(ga, id % ga.obQ, id / ga.obQ, gsmem);
  } else {
    const int t = id - nQ;
    grad128_body<false, SYM>(ga, t % ga.obP, t / ga.obP, gsmem);
  }
}

// ===========================================================================
// Statistics pass for d = 128 (Eq. 4's normaliser, the positive's logit and the arg-max, per anchor and split).
// The layout of the d = 128 gradient pass without its second contraction: a workgroup (4 waves) owns 256 anchors,
// each wave 64 of them with all 128 columns in registers, and all four share the streamed target tiles (32 rows)
// through the same LDS ring.  Lane (n, h) holds, for its two anchors 32 i + n, the scores of 16 of a tile's 32
// targets; the other 16 are in lane (n, h ^ 1).  The running (max, sum, arg-max) of an anchor therefore lives in
// a lane of its own and no lane talks to another before the end of the stream: 16 MFMAs against about 5 vector
// operations per score, which a second workgroup on the same CU runs behind the first one's MFMAs.
// ===========================================================================
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
  const int a0 = ablk * G1_OWN + w * G1_OWN_W;   // this wave's first anchor
  const int sbeg = split * cols_per_split, send = min(P, sbeg + cols_per_split);
  const int nt = (send - sbeg + G1_T - 1) / G1_T;   // >= 1
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
  const unsigned voff_full[2] = {src_of(2 * w, G1_T - 1), src_of(2 * w + 1, G1_T - 1)};
  auto prefetch = [&](int u) __attribute__((always_inline)) {
    const int t0 = sbeg + u * G1_T;
    const unsigned st = lds0 + (u & (G1_STAGES - 1)) * G1_STAGE;
    const unsigned short* tile = Pm + (size_t)t0 * D;
    if (t0 + G1_T <= P) {
      dma_group<1>(tile, &voff_full[0], st + G1_STAT + (2 * wu) * 1024);
      dma_group<1>(tile, &voff_full[1], st + G1_STAT + (2 * wu + 1) * 1024);
    } else {  // ragged last tile: rows past the end re-read the last valid row (masked below)
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const unsigned off = src_of(2 * w + k, P - 1 - t0);
        dma_group<1>(tile, &off, st + G1_STAT + (2 * wu + k) * 1024);
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
    const unsigned char* st = s1mem + (u & (G1_STAGES - 1)) * G1_STAGE;
    const int t0 = sbeg + u * G1_T;

    bf16x8 pfr[8];
#pragma unroll
    for (int k = 0; k < 8; k++) pfr[k] = *(const bf16x8*)(st + G1_STAT + ln * 256 + (((2 * k + h) ^ (int)sw_ln) * 16));
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
    bool rare = (t0 + G1_T > send) || (mask_self && t0 < a0 + G1_OWN_W && t0 + G1_T > a0);
    rare = rare || (unsigned)(r_o[0] - t0) < (unsigned)G1_T || (unsigned)(r_o[1] - t0) < (unsigned)G1_T;
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

template <bool ARGMAX>
static hipError_t stats128_launch(const LossArgs& a, const LossPlan& pl) {
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)stats128_kernel<ARGMAX>, G1_SMEM, attr_done); e != hipSuccess) return e;
  char* ws = a.ws;
  const int n_ablk = (a.B + G1_OWN - 1) / G1_OWN;
  stats128_kernel<ARGMAX><<<n_ablk * pl.stat_splits, 256, G1_SMEM, a.stream>>>(
      (const unsigned short*)a.q, (const unsigned short*)a.p, a.pos_idx, a.B, a.P, a.alpha * kLog2e,
      (a.flags & GC_MASK_SELF) ? 1 : 0, n_ablk, pl.stat_cols_per_split, (float*)(ws + pl.off_part_m),
      (float*)(ws + pl.off_part_l), (int*)(ws + pl.off_part_idx), (float*)(ws + pl.off_pos));
  return hipGetLastError();
}
hipError_t launch_stats128(const LossArgs& a, const LossPlan& pl) {
  return a.argmax ? stats128_launch<true>(a, pl) : stats128_launch<false>(a, pl);
}

template <bool SYM>
static hipError_t grad128_launch_as(const GradArgs& ga, int nwg, hipStream_t stream) {
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)grad128_kernel<SYM>, G1_SMEM, attr_done); e != hipSuccess) return e;
  grad128_kernel<SYM><<<nwg, 256, G1_SMEM, stream>>>(ga);
  return hipGetLastError();
}

hipError_t grad128_launch(const GradArgs& ga, int nwg, hipStream_t stream) {
  return ga.lse2_t ? grad128_launch_as<true>(ga, nwg, stream) : grad128_launch_as<false>(ga, nwg, stream);
}

}  // namespace gc
