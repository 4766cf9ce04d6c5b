// Gradient walks of the bf16 loss path for gfx950, widths from 256 (d = 128: loss_mfma128.hip).
//
//   gradient pass  Eq. 5 / Eq. 6: a workgroup owns 64 rows of dQ (or dP), streams the other
//                matrix, recomputes the score tile, forms g = softmax - Y in registers and
//                accumulates g * rows with MFMA.
// (The kernels: loss_mfma.hip, and loss_mfma_sym.hip for the symmetric forms.)
#pragma once
#include "mfma_common.h"

namespace gc {

// ===========================================================================
// Gradient pass.  Workgroup = 256 threads = 4 waves, one per SIMD (up to 512 registers a lane).
// It owns 64 rows of the output (dQ rows: "owner" = Q, streamed = P; dP rows: owner = P,
// streamed = Q) and walks the streamed matrix 16 rows at a time:
//   phase 1  S^T tile [16 streamed x 64 owner] = R_tile * O^T (v_mfma_f32_16x16x32_bf16).  The
//            contraction over d is split four ways over the waves (wave w takes columns
//            [w*D/4, (w+1)*D/4)), so that each wave keeps its slice of the owner rows in
//            registers for the whole kernel and only ever touches its own D/4-column slice of
//            every streamed tile (a wave-private LDS ring of five stages, filled by direct
//            global->LDS loads issued four tiles ahead: the loads of iteration u go to the stage
//            that iteration u-1 has finished with, so they can sit anywhere in the iteration).
//   exchange the four partial tiles are summed through LDS (each wave finishes 16 owner rows, in
//            a fixed order), turned into g = 2^(t - lse2) - [j = r_i] (Eq. 5 / Eq. 6 with eps_j
//            of Eq. 7 folded in), rounded to bf16 and published as ready-made MFMA A fragments.
//   phase 2  dO[64 x D/4 slice] += g[64 x 16] * R_tile[16 x D/4 slice] (v_mfma_f32_32x32x16_bf16);
//            the streamed slice is read back from the same LDS stage with transposing loads
//            (ds_read_b64_tr_b16).
// The three steps of consecutive tiles are software-pipelined so that one workgroup barrier per
// tile suffices: iteration u publishes the partials of tile u+1 and the fragments of tile u,
// then runs phase 1 of tile u+2 and phase 2 of tile u while the exchanged data is in flight.
//
// 16x16x32 layouts: A lane l holds A[m = l % 16][k = 8 * (l / 16) + 0..7], B likewise with n,
// D register r of lane l holds D[m = 4 * (l / 16) + r][n = l % 16].
// ds_read_b64_tr_b16: in each group of 16 lanes, lane j supplies the address of 4 consecutive
// 16-bit elements; lane i receives element (i % 4) of the addresses of lanes i / 4 + {0, 4, 8, 12}.
// ===========================================================================
constexpr int GR_OWN = 64, GR_T = 16, GR_STAGES = 5;
// The loops of the four waves of the widest kernels are more code than an instruction cache holds, and where they start moves the
// headline call by 1.5 %: 4096 x 8192 x 768 245 us with the kernels at multiples of 8 KB, 247 with the same code 4 KB off.
#define GR_CODE_ALIGN __attribute__((aligned(8192)))

template <int D>
struct GradCfg {
  static constexpr int DS = D / 4;        // columns per wave
  static constexpr int KS = DS / 32;      // MFMA k-steps of phase 1 (k = 32 each)
  static constexpr int CT = DS / 32;      // 32-column output tiles of phase 2
  static constexpr int C16 = DS / 8;      // 16-byte chunks per slice row
  // LDS layout of a streamed slice: 16 rows of C16 chunks.  When C16 = 8 (mod 16) the rows are
  // stored unpadded with the low three bits of the chunk index XORed by swz3(row): the 16 rows
  // of a phase-1 fragment read and the 4 rows x 4 chunks of a transposing phase-2 read then fall
  // into 16 different 16-byte bank groups.  Other widths keep one pad chunk per row instead.
  static constexpr bool SWZ = (C16 % 16) == 8;
  static constexpr int SLOTS = SWZ ? C16 : C16 + 1;
  static constexpr int LDB = SLOTS * 16;                // LDS row stride in bytes
  static constexpr int TILE_SLOTS = GR_T * SLOTS;       // 16-byte slots holding tile data
  static constexpr int NI_Q = (TILE_SLOTS + 63) / 64;   // direct-to-LDS load instructions (1 KB each) per tile slice
  // a stage starts with the row statistics of the streamed rows (dP role): 64 bytes of lse2, then
  // 64 bytes of pos_idx; the tile data follows
  static constexpr int TOFF = 128;
  static constexpr int STAGE = TOFF + NI_Q * 1024;      // bytes: one wave, one stage
  static constexpr int RS_BYTES = 4 * GR_STAGES * STAGE;
  static constexpr int X_BYTES = 2 * 4 * 4 * 64 * 16;   // [parity][src][dst][lane] float4
  static constexpr int G_BYTES = 2 * 2 * 64 * 16;       // [parity][m-tile][lane] bf16x8
  // online-statistics walk: [parity][64 rescale factors (float) | 4 flag words, one per finishing wave]
  static constexpr int F_PAR = 64 * 4 + 16;
  static constexpr int F_BYTES = 1024;
  static constexpr int SMEM = RS_BYTES + X_BYTES + G_BYTES + F_BYTES;
  static_assert(SMEM <= 160 * 1024, "LDS budget");
};

// (Measured with the bank-conflict counter on the two read patterns, all 4096 linear maps of the row bits: this one
// and 767 others are free of conflicts for both; the first choice, bits 2 and 3 of the row into bits 0 and 1, left
// the 16-byte fragment reads of phase 1 with a two-way conflict, 21 % of the walks' LDS cycles.)
__device__ __forceinline__ int swz3(int row) { return (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1); }

template <int D>
constexpr bool grad_offsets_fit() {  // voff[k] - 1024 (k % 4) must stay >= 0 for a full tile
  using C = GradCfg<D>;
  for (int it = 0; it < C::NI_Q; it++)
    if ((64 * it / C::SLOTS) * 2 * D < (it & 3) * 1024) return false;
  return true;
}

// SYM: the symmetric loss 1/2 [L(F, G, r) + L(G, F, r^-1)].  Its coefficient matrix is
//   g_ij = 1/2 (2^(t_ij - lse2[i]) + 2^(t_ij - lse2_t[j])) - [j = r_i]
// (row softmax and column softmax of the same scores), and dQ = g P, dP = g^T Q as before: one walk per side,
// in which the streamed rows always bring their statistic along.  ONE_EXP: one exponential a score (see kWideLse), both
// statistics as wexp.  Forms of their own, so that neither pays for the other: with the second form's two exponentials behind
// a branch of the first, beside its own, the calls whose logits are beyond kWideLse took 4 to 12 % longer (symmetric loss 8192 x 384
// 419 us, 394 so and 374 in the first form; NT-Xent 8192 x 256 153, 144 so).
// ONLINE (dQ role only): no statistics pass has run.  The walk keeps, per owner row, a reference m (the row
// maximum of the first tile; raised, with the accumulators and the running sum rescaled by 2^(old - new), only when
// a later score exceeds it by more than kOnlineMargin), accumulates sum_j 2^(t_ij - m) p_j and sum_j 2^(t_ij - m),
// and tracks the true maximum, its first index and the positive's logit.  A later kernel turns these into lse2 and
// dQ (softmax_ij = 2^(t_ij - m) 2^(m - lse2_i); the positive's -p_{r_i} is subtracted there).
constexpr float kOnlineMargin = 16.f;
template <int D, bool OWNER_IS_Q, bool SYM, bool ONLINE = false, bool ONE_EXP = false>
__device__ __forceinline__ void grad_body(const GradArgs& ga, int oblk, int split, unsigned char* smem) {
  using C = GradCfg<D>;
  static_assert(!ONLINE || (OWNER_IS_Q && !SYM), "the online walk is the dQ role of the one-direction loss");
  static_assert(!ONE_EXP || SYM, "see kWideLse");
  constexpr bool STR_STATS = SYM || !OWNER_IS_Q;   // the streamed rows' statistics ride in the LDS stage
  const float* stat_q = ONE_EXP ? ga.wexp : ga.lse2;
  const float* stat_p = ONE_EXP ? ga.wexp_t : ga.lse2_t;
  const float* lse_own = (SYM && !OWNER_IS_Q) ? stat_p : stat_q;
  const float* lse_str = (SYM && OWNER_IS_Q) ? stat_p : stat_q;
  static_assert(grad_offsets_fit<D>(), "direct-to-LDS load offsets");
  int tid = threadIdx.x;
  // what follows from the thread's index is then not shared between the two forms (768: 47 registers spilled if it is)
  if constexpr (SYM) asm volatile("" : "+v"(tid));
  const int lane = tid & 63, w = tid >> 6, h = lane >> 5, ln = lane & 31;
  const int l16 = lane & 15, g16 = lane >> 4;
  const unsigned short* O = OWNER_IS_Q ? ga.Q : ga.P;
  const unsigned short* R = OWNER_IS_Q ? ga.P : ga.Q;
  const int No = OWNER_IS_Q ? ga.B : ga.Pn, Nr = OWNER_IS_Q ? ga.Pn : ga.B;
  const int slen = OWNER_IS_Q ? ga.q_stream_len : ga.p_stream_len;
  const int a0 = oblk * GR_OWN;
  const int sbeg = split * slen, send = min(Nr, sbeg + slen);
  const int nt = (send - sbeg + GR_T - 1) / GR_T;  // streamed tiles of this workgroup (>= 1)

  // ---- LDS map (bytes): [wave rings: 4 waves x 5 stages x STAGE][X: 2 x 4 x 4 x 1024][G: 2 x 2 x 1024]
  constexpr int NT = C::NI_Q;                                 // load instructions that carry tile data
  constexpr unsigned RING = GR_STAGES * C::STAGE;
  const unsigned ring_off = w * RING;                         // this wave's ring of stages
  const unsigned ring_m0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)smem + ring_off);
  // per-lane byte offsets; every access adds the stage offset and a compile-time constant (k-step ...)
  auto lane_base = [&](int row, int j, int parity) __attribute__((always_inline)) -> unsigned {
    // chunk 4 i + j of a row is stored at 4 (i ^ s2) + (j ^ s01), (s2, s01) from swz3(row): one
    // base for even i and one for odd i, the loops add the compile-time part 64 i
    const int sw = C::SWZ ? swz3(row) : 0;
    const int s2 = sw >> 2, s01 = sw & 3;
    return ring_off + C::TOFF + (unsigned)(row * C::LDB + 16 * (j ^ s01) + (parity ? -64 * s2 : 64 * s2));
  };
  // phase 1 reads row l16, chunk 4 ks + g16
  const unsigned char* p1p[2] = {smem + lane_base(l16, g16, 0), smem + lane_base(l16, g16, 1)};
  // phase 2 (transposing read): rows 8 h + l16 / 4 (+4), chunk 4 ct + 2 (g16 & 1) + (lane & 3) / 2, 8 bytes
  const int tr_row = 8 * h + (l16 >> 2), tr_j = 2 * (g16 & 1) + ((lane & 3) >> 1), tr_in = 8 * (lane & 1);
  const unsigned char* p2lo[2] = {smem + lane_base(tr_row, tr_j, 0) + tr_in, smem + lane_base(tr_row, tr_j, 1) + tr_in};
  const unsigned char* p2hi[2] = {smem + lane_base(tr_row + 4, tr_j, 0) + tr_in, smem + lane_base(tr_row + 4, tr_j, 1) + tr_in};
  unsigned char* xwp = smem + C::RS_BYTES + (w * 4) * 1024 + lane * 16;          // + par * 16384 + dst * 1024
  const unsigned char* xrp = smem + C::RS_BYTES + w * 1024 + lane * 16;          // + par * 16384 + src * 4096
  // lane (w, l16, g16) finishes rows 4 g16 + 0..3 of owner row 16 w + l16: half (g16 & 1) of the A fragment
  // elements of lane 16 (w & 1) + l16 + 32 (g16 >> 1) in m-tile w >> 1
  unsigned char* gwp = smem + C::RS_BYTES + C::X_BYTES + ((w >> 1) * 64 + 16 * (w & 1) + l16 + 32 * (g16 >> 1)) * 16 + 8 * (g16 & 1);
  const unsigned char* grp = smem + C::RS_BYTES + C::X_BYTES + lane * 16;        // + par * 2048 + mt * 1024
  const unsigned char* rip = smem + ring_off + 16 * g16;                         // + stage offset (+ 64: pos_idx)

  // owner slice, kept in registers as MFMA B fragments of phase 1 (16 owner rows per fragment)
  bf16x8 ofrag[4][C::KS];
#pragma unroll
  for (int nq = 0; nq < 4; nq++) {
    const int row = min(a0 + 16 * nq + l16, No - 1);
#pragma unroll
    for (int ks = 0; ks < C::KS; ks++)
      ofrag[nq][ks] = *(const bf16x8*)(O + (size_t)row * D + w * C::DS + 32 * ks + 8 * g16);
  }
  // this wave finishes the scores of owner rows 16 w .. 16 w + 15; a lane holds streamed rows 4 * g16 + 0..3
  const int a_q = a0 + 16 * w + l16;
  float lse_a = 0.f; int r_a = -1;
  if ((OWNER_IS_Q || SYM) && !ONLINE) lse_a = lse_own[a_q];   // padded: +inf past the end, so g = 0 there
  if (OWNER_IS_Q && !ONLINE) r_a = ga.pos_pad[a_q];
  if (ONLINE) r_a = (a_q < No) ? ga.pos_pad[a_q] : -1;   // here pos_pad is the caller's pos_idx itself (B entries)

  // ---- direct-to-LDS loads of a streamed tile: slot q = it * 64 + lane -> (row, chunk) -------------------------
  auto slot_src = [&](int q, int max_row) __attribute__((always_inline)) -> unsigned {
    const int row = min(min(q / C::SLOTS, GR_T - 1), max_row);
    int c = min(q % C::SLOTS, C::C16 - 1);
    if (C::SWZ) c ^= swz3(row);
    return (unsigned)((row * D + w * C::DS + c * 8) * 2);
  };
  unsigned src_off[NT];  // full tile, with the instruction offset 1024 (it % 4) pre-subtracted
#pragma unroll
  for (int it = 0; it < NT; it++) src_off[it] = slot_src(it * 64 + lane, GR_T - 1) - 1024u * (it & 3);
  // row statistics of the streamed rows: lanes 0-3 load lse_str[t0 + 4 l ..], lanes 4-7 pos_pad (dP role; in
  // the dQ role of the symmetric loss they load the same as lanes 0-3 and nobody reads it)
  const unsigned ri_off = ((lane & 4) && !OWNER_IS_Q) ? (unsigned)((const char*)ga.pos_pad - (const char*)lse_str) + 16u * (lane & 3) : 16u * (lane & 3);
  constexpr int NI = STR_STATS ? NT + 1 : NT;  // load instructions per tile
  // piece k (0 .. NI-1) of the loads of a full tile that starts at row t0, into the stage at byte offset so
  auto prefetch_piece = [&](auto k_tag, auto two_tag, int t0, unsigned so, u32x4& pin_a, u32x4& pin_b) __attribute__((always_inline)) {
    constexpr int K = decltype(k_tag)::value;
    constexpr bool TWO = decltype(two_tag)::value;
    if constexpr (STR_STATS && K == 0) {
      dma_piece_pinned<0, true, TWO>(lse_str + t0, ri_off, ring_m0 + so, pin_a, pin_b);
    } else {
      constexpr int IT = STR_STATS ? K - 1 : K;
      dma_piece_pinned<1024 * (IT & 3), false, TWO>(R + (size_t)t0 * D, src_off[IT], ring_m0 + so + C::TOFF + 4096 * (IT >> 2), pin_a, pin_b);
    }
  };
  auto prefetch = [&](int u, unsigned so) __attribute__((always_inline)) {  // whole tile u -> stage at offset so
    const int t0 = sbeg + u * GR_T;
    const unsigned short* tile = R + (size_t)t0 * D;  // wave-uniform
    const unsigned lds0 = ring_m0 + so + C::TOFF;
    if (STR_STATS) {
      if (lane < 8) dma_piece<0>(lse_str + t0, ri_off, ring_m0 + so);
    }
    if (t0 + GR_T <= Nr) {
#pragma unroll
      for (int g = 0; g < NT; g += 4) {
        if (NT - g >= 4) dma_group<4>(tile, &src_off[g], lds0 + g * 1024);
        else if (NT - g == 3) dma_group<3>(tile, &src_off[g], lds0 + g * 1024);
        else if (NT - g == 2) dma_group<2>(tile, &src_off[g], lds0 + g * 1024);
        else dma_group<1>(tile, &src_off[g], lds0 + g * 1024);
      }
    } else {  // ragged last tile: rows past the end re-read the last valid row (their g is forced to 0)
#pragma unroll
      for (int it = 0; it < NT; it++) {
        const unsigned off = slot_src(it * 64 + lane, Nr - 1 - t0);
        dma_group<1>(tile, &off, lds0 + it * 1024);
      }
    }
  };

  f32x16 acc[2][C::CT];
#pragma unroll
  for (int mt = 0; mt < 2; mt++)
#pragma unroll
    for (int ct = 0; ct < C::CT; ct++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[mt][ct][r] = 0.f;

  f32x4 sacc[4];  // partial S^T of the tile most recently through phase 1: [owner 16-block]
  u32x4 afr[C::KS];  // phase-1 A fragments of the tile being started (bf16x8 each)
  auto p1_load = [&](unsigned so, int ks0, int ks1) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = ks0; ks < ks1; ks++) afr[ks] = *(const u32x4*)(p1p[ks & 1] + so + 64 * ks);
  };
  auto p1_mfma = [&](int ks0, int ks1) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = ks0; ks < ks1; ks++)
#pragma unroll
      for (int nq = 0; nq < 4; nq++)
        sacc[nq] = mfma16(__builtin_bit_cast(bf16x8, afr[ks]), ofrag[nq][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sacc[nq]);
  };
  // The load unit of a compute unit takes one 1 KB load every 16 cycles, and a wave waits at the load
  // until the unit accepts it.  The four waves run in step (one barrier per tile), so a steady iteration
  // spreads its 4 NI loads evenly over the MFMA time of the iteration and the waves take turns: the code
  // of the steady loop is specialised per wave (WAVE = 0 .. 3), piece k of wave WAVE follows the MFMA
  // that runs at 1 / (4 NI) * (4 k + WAVE) of that time.  Sections: 0 = phase 1 before the barrier,
  // 1 = phase 1 after it, 2 = phase 2.
  constexpr int KS_PRE = (C::KS + 1) / 2;            // k-steps of phase 1 issued before the barrier
  static_assert(C::KS == C::CT, "the steady loop pairs the k-steps of phase 1 with the column tiles of phase 2");
  constexpr int MA = 4 * KS_PRE, MB = 4 * (C::KS - KS_PRE), MC = 2 * C::CT;  // MFMAs per section
  constexpr int T16 = 19, T32 = 33;                  // measured issue-to-issue cycles of the two MFMA shapes
  auto slot_of = [](int wave, int k, int sec) constexpr -> int {  // MFMA index in section sec, or -1
    constexpr int TOTAL = T16 * (MA + MB) + T32 * MC;
    int t = ((4 * k + wave) * TOTAL) / (4 * NI);
    if (t < T16 * MA) return sec == 0 ? t / T16 : -1;
    t -= T16 * MA;
    if (t < T16 * MB) return sec == 1 ? t / T16 : -1;
    t -= T16 * MB;
    return sec == 2 ? (t / T32 < MC ? t / T32 : MC - 1) : -1;
  };
  // loads of tile u+4 that a steady iteration of wave `wave` has issued once the round of phase-2 MFMA `idx` is over
  auto issued_by = [slot_of](int wave, int idx) constexpr -> int {
    int n = 0;
    for (int k = 0; k < NI; k++) {
      const int s2 = slot_of(wave, k, 2);
      if (slot_of(wave, k, 0) >= 0 || slot_of(wave, k, 1) >= 0 || (s2 >= 0 && s2 <= idx)) n++;
    }
    return n;
  };
  // called after MFMA number IDX of section SEC; pin_a: a register that MFMA read, pin_b: one that the
  // next MFMA reads (TWO: they differ)
  auto spread = [&](auto wave_tag, auto sec_tag, auto idx_tag, auto two_tag, int t_pf, unsigned so_pf, u32x4& pin_a, u32x4& pin_b) __attribute__((always_inline)) {
    constexpr int WAVE = decltype(wave_tag)::value, SEC = decltype(sec_tag)::value, IDX = decltype(idx_tag)::value;
    if constexpr (WAVE >= 0) {
      static_for<NI>([&](auto k_tag) __attribute__((always_inline)) {
        if constexpr (slot_of(WAVE, decltype(k_tag)::value, SEC) == IDX) prefetch_piece(k_tag, two_tag, t_pf, so_pf, pin_a, pin_b);
      });
    }
  };
  // phase 2 of the tile in the stage at `so` (WAVE >= 0: a steady iteration, which also issues its share
  // of the loads of the tile that starts at row t_pf into the stage at so_pf)
  u32x4 bfr[C::CT];  // phase-2 B fragments (bf16x8 each)
  auto p2_load = [&](unsigned so, int c0, int c1) __attribute__((always_inline)) {
#pragma unroll
    for (int ct = c0; ct < c1; ct++) {
      s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p2lo[ct & 1] + so + 64 * ct));
      s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p2hi[ct & 1] + so + 64 * ct));
      s16x8 bb = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      bfr[ct] = __builtin_bit_cast(u32x4, bb);
    }
  };
  // The LDS pipe is shared by the four waves, which run in step: fragment reads bunched at the start of a phase
  // leave the MFMAs waiting for LDS and LDS idle during the MFMAs.  A steady iteration therefore reads every fragment
  // half an iteration ahead, into the registers of a fragment that has just been used up: the transposed fragment ct
  // of phase 2 (tile u, stage so_p2) right behind the four MFMAs of k-step ct of phase 1, and the fragment of k-step ks
  // of the NEXT iteration's phase 1 (tile u+3, stage so_p1n) right behind the two MFMAs of column tile ks of phase 2.
  auto p1_mfma_spread = [&](auto wave_tag, auto sec_tag, int t_pf, unsigned so_pf, unsigned so_p2) __attribute__((always_inline)) {
    constexpr int SEC = decltype(sec_tag)::value, WAVE = decltype(wave_tag)::value;
    constexpr int KS0 = SEC == 0 ? 0 : KS_PRE, KS1 = SEC == 0 ? KS_PRE : C::KS;
    static_for<4 * (KS1 - KS0)>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value, ks = KS0 + i / 4, nq = i % 4;
      sacc[nq] = mfma16(__builtin_bit_cast(bf16x8, afr[ks]), ofrag[nq][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sacc[nq]);
      constexpr int ksn = KS0 + (i + 1) / 4;  // k-step of the next MFMA of the section
      if constexpr (ksn != ks && ksn < KS1) spread(wave_tag, sec_tag, i_tag, std::true_type{}, t_pf, so_pf, afr[ks], afr[ksn]);
      else spread(wave_tag, sec_tag, i_tag, std::false_type{}, t_pf, so_pf, afr[ks], afr[ks]);
      if constexpr (WAVE >= 0 && nq == 3) p2_load(so_p2, ks, ks + 1);
    });
  };
  // after_round(i): arithmetic of the caller that is to run in the shadow of MFMA i
  auto phase2 = [&](const bf16x8 (&gf)[2], auto wave_tag, int t_pf, unsigned so_pf, unsigned so_p1n, auto&& after_round) __attribute__((always_inline)) {
    constexpr int WAVE = decltype(wave_tag)::value;
    static_for<MC>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value, ct = i / 2, mt = i % 2;
      acc[mt][ct] = mfma32(gf[mt], __builtin_bit_cast(bf16x8, bfr[ct]), acc[mt][ct]);
      constexpr std::integral_constant<int, 2> sec{};
      if constexpr (mt == 1 && ct + 1 < C::CT) spread(wave_tag, sec, i_tag, std::true_type{}, t_pf, so_pf, bfr[ct], bfr[ct + 1]);
      else spread(wave_tag, sec, i_tag, std::false_type{}, t_pf, so_pf, bfr[ct], bfr[ct]);
      if constexpr (WAVE >= 0 && mt == 1) {
        // tile u+3 has landed once at most the loads this iteration has issued so far (for tile u+4) are in flight
        if constexpr (ct == 0) wait_vmem<issued_by(WAVE, i)>();
        p1_load(so_p1n, ct, ct + 1);
      }
      after_round(i_tag);
    });
  };

  bf16x4 gq = {0, 0, 0, 0};  // g of the tile whose scores were finished last (4 streamed rows of owner row a_q)
  // online walk: state of owner row a_q (m_run is the same in the four lanes that share the row, the rest is per lane)
  float m_run = -INFINITY, l_run = 0.f, best_v = -INFINITY, f_pub = 1.f;
  int best_i = 0x7fffffff, need_pub = 0;
  unsigned char* fwp = smem + C::RS_BYTES + C::X_BYTES + C::G_BYTES;            // + par * F_PAR

  // One pipeline iteration (see the header comment); so0 = ring offset of the stage of tile u.  STEADY:
  // every pipeline slot is live, the tiles involved are full and not the last ones.
  // STG >= 0: the ring stage of tile u is known at compile time (the steady loop is unrolled over the five stages), so
  // every LDS address of the iteration is a per-lane base plus an immediate and no address arithmetic is issued: a
  // single wave per SIMD issues everything itself, and what it issues besides the MFMAs is what the loop's time is made of.
  auto body = [&](int u, unsigned so0_dyn, auto stage_tag, auto wave_tag) __attribute__((always_inline)) {
    constexpr int WAVE = decltype(wave_tag)::value, STG = decltype(stage_tag)::value;
    constexpr bool STEADY = WAVE >= 0;
    const unsigned so0 = STG >= 0 ? (unsigned)(STG * C::STAGE) : so0_dyn;
    const int t_pf = sbeg + (u + 4) * GR_T;  // first row of tile u+4
    const unsigned so1 = (so0 + C::STAGE >= RING) ? so0 + C::STAGE - RING : so0 + C::STAGE;   // tile u+1
    const unsigned so2 = (so1 + C::STAGE >= RING) ? so1 + C::STAGE - RING : so1 + C::STAGE;   // tile u+2
    const unsigned so4 = (so0 == 0) ? RING - C::STAGE : so0 - C::STAGE;                        // tile u+4 (= u-1)
    const int PAR0 = u & 1, PAR1 = PAR0 ^ 1;           // X / G parity of tiles u and u+1
    const bool xw = STEADY || (u + 1 < nt);            // tile u+1: publish partials, finish scores
    const bool gw = STEADY || (u >= 0);                // tile u: publish fragments, phase 2   (u < nt always)
    const bool p1 = STEADY || (u + 2 < nt);            // tile u+2: phase 1
    const bool pf = STEADY || (u >= 0 && u + 4 < nt);  // tile u+4: start its loads
    __builtin_amdgcn_iglp_opt(0);  // scheduler hint: interleave the LDS reads with the MFMA stream
    if (p1 && !STEADY) {
      // tile u+2 has landed; its fragment reads are issued ahead of the writes below, so they come back first.  (A
      // steady iteration finds them in registers: the iteration before it has read them during its phase 2.)
      wait_vmem<0>();
      p1_load(so2, 0, C::KS);
    }
    // the partial tile of the owner rows this wave finishes itself stays in registers (steady loop: the wave
    // index is a compile-time constant there); the other three go through LDS
    f32x4 own = {0.f, 0.f, 0.f, 0.f};
    if constexpr (STEADY) own = sacc[WAVE];
    if (xw) {
#pragma unroll
      for (int dst = 0; dst < 4; dst++)
        if (!(STEADY && dst == WAVE)) *(f32x4*)(xwp + PAR1 * 16384 + dst * 1024) = sacc[dst];
    }
    if (gw) *(bf16x4*)(gwp + PAR0 * 2048) = gq;
    if (ONLINE && gw) {  // the rescale factors of tile u's rows and this wave's "some row was rescaled" word
      if (g16 == 0) *(float*)(fwp + PAR0 * C::F_PAR + (16 * w + l16) * 4) = f_pub;
      if (lane == 0) *(int*)(fwp + PAR0 * C::F_PAR + 256 + 4 * w) = need_pub;
    }
    if (p1) p1_mfma_spread(wave_tag, std::integral_constant<int, 0>{}, t_pf, so4, so0);  // while the writes drain and the barrier gathers the waves
    __syncthreads();
    f32x4 xr[4];
    if (xw) {
#pragma unroll
      for (int src = 0; src < 4; src++) {
        if (STEADY && src == WAVE) xr[src] = own;
        else xr[src] = *(const f32x4*)(xrp + PAR1 * 16384 + src * 4096);
      }
    }
    bf16x8 gf[2];
    if (gw) {
#pragma unroll
      for (int mt = 0; mt < 2; mt++) gf[mt] = *(const bf16x8*)(grp + PAR0 * 2048 + mt * 1024);
    }
    f32x4 lse_r = {0.f, 0.f, 0.f, 0.f}; i32x4 pos_r = {0, 0, 0, 0};
    if (STR_STATS && xw) {  // row statistics of tile u+1 ride in its LDS stage
      lse_r = *(const f32x4*)(rip + so1);
      if (!OWNER_IS_Q) pos_r = *(const i32x4*)(rip + so1 + 64);
    }
    i32x4 fl = {0, 0, 0, 0};
    if (ONLINE && gw) fl = *(const i32x4*)(fwp + PAR0 * C::F_PAR + 256);
    if (p1) p1_mfma_spread(wave_tag, std::integral_constant<int, 1>{}, t_pf, so4, so0);
    if constexpr (ONLINE) __builtin_amdgcn_sched_barrier(0);  // the flag test (and its wait for LDS) stays behind these MFMAs
    if (!STEADY && gw) p2_load(so0, 0, C::CT);   // (a steady iteration has read them behind the MFMAs of phase 1)
    if (ONLINE && gw) {
      // rare after the first tile: some row's reference went up, every wave rescales its columns of those rows
      if (__builtin_amdgcn_ballot_w64((fl[0] | fl[1] | fl[2] | fl[3]) != 0) != 0) {
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
          for (int j = 0; j < 4; j++) {
            const f32x4 f4 = *(const f32x4*)(fwp + PAR0 * C::F_PAR + (32 * mt + 8 * j + 4 * h) * 4);
#pragma unroll
            for (int ct = 0; ct < C::CT; ct++)
#pragma unroll
              for (int i = 0; i < 4; i++) {
                // in place on the accumulation register (written in the compiler's own way this cold path moved
                // every accumulator into ordinary registers and cost the loop 200 spilled ones); the MFMAs that
                // wrote and will read these registers are a barrier and many instructions away
                float x = acc[mt][ct][4 * j + i], tmp;
                asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1"
                             : "+a"(x), "=&v"(tmp) : "v"(f4[i]));
                acc[mt][ct][4 * j + i] = x;
              }
          }
      }
    }
    // ---- from the summed scores of tile u+1 to its coefficients.  The arithmetic that every tile needs is cut into
    // pieces; in a steady iteration piece k runs right behind MFMA k * MC / NP of phase 2, where a
    // wave's own arithmetic is free, instead of after the last MFMA, where it is not.  What only few tiles need
    // (the positive, masks, the arg-max) stays behind phase 2.
    constexpr bool INTER = STEADY && (!SYM || ONE_EXP);   // (two exponentials a score: 8192 x 640, 554 us a call interleaved, 524 not)
    constexpr int NP = ONLINE ? 10 : SYM && !ONE_EXP ? 6 : 5;
    const int b0 = sbeg + (u + 1) * GR_T + 4 * g16;      // first of this lane's 4 streamed rows
    f32x4 sv = {0.f, 0.f, 0.f, 0.f}, tt = {0.f, 0.f, 0.f, 0.f}, gv = {0.f, 0.f, 0.f, 0.f};
    float tmx = 0.f, mref = 0.f;
    bool need = false;
    auto piece = [&](auto k_tag) __attribute__((always_inline)) {
      constexpr int K = decltype(k_tag)::value;
      if constexpr (K == 0) sv = xr[0] + xr[1];            // fixed order ((x0 + x1) + x2) + x3: bit-identical
      else if constexpr (K == 1) sv = sv + xr[2];           // whichever wave sums
      else if constexpr (K == 2) sv = sv + xr[3];
      else if constexpr (!ONLINE) {
        if constexpr (K == 3) {
#pragma unroll
          for (int e = 0; e < 4; e++) tt[e] = SYM ? sv[e] * ga.alpha2 : sv[e] * ga.alpha2 - (OWNER_IS_Q ? lse_a : lse_r[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; e++) {
            if constexpr (!SYM) gv[e] = fast_exp2(tt[e]);   // softmax
            else if constexpr (ONE_EXP) gv[e] = fast_exp2(tt[e]) * (lse_a + lse_r[e]);
            else if constexpr (K == 4) gv[e] = fast_exp2(tt[e] - (lse_a + 1.f));   // mean of the row softmax and ...
            else gv[e] += fast_exp2(tt[e] - (lse_r[e] + 1.f));                      // ... the column softmax
          }
        }
      } else {
        if constexpr (K == 3) {
#pragma unroll
          for (int e = 0; e < 4; e++) tt[e] = sv[e] * ga.alpha2;
          if constexpr (!STEADY) {  // rows past the end of the split, the diagonal under mask_self
            const int t1o = b0 - 4 * g16;
            if ((t1o + GR_T > send) || (ga.mask_self && (t1o < a0 + GR_OWN) && (t1o + GR_T > a0))) {
#pragma unroll
              for (int e = 0; e < 4; e++)
                if (b0 + e >= send || (ga.mask_self && b0 + e == a_q)) tt[e] = -INFINITY;
            }
          }
        } else if constexpr (K == 4) tmx = fmaxf(fmaxf(tt[0], tt[1]), fmaxf(tt[2], tt[3]));
        else if constexpr (K == 5) {
          unsigned x0, x1;
          swap16(__builtin_bit_cast(unsigned, tmx), x0, x1);
          tmx = fmaxf(__builtin_bit_cast(float, x0), __builtin_bit_cast(float, x1));
        } else if constexpr (K == 6) {
          unsigned x0, x1;
          swap32(__builtin_bit_cast(unsigned, tmx), x0, x1);
          tmx = fmaxf(__builtin_bit_cast(float, x0), __builtin_bit_cast(float, x1));   // this tile's maximum of row a_q
        } else if constexpr (K == 7) {
          // raise the reference when the tile exceeds it by more than the margin (always at the first tile with a
          // finite score: m_run = -inf); without branches: the factor is 2^0 when nothing changes, 2^-inf the first time
          need = tmx > m_run + kOnlineMargin;
          f_pub = fast_exp2(need ? m_run - tmx : 0.f);
          l_run *= f_pub;
          m_run = need ? tmx : m_run;
          mref = (m_run == -INFINITY) ? 0.f : m_run;
        } else if constexpr (K == 8) {
#pragma unroll
          for (int e = 0; e < 4; e++) gv[e] = fast_exp2(tt[e] - mref);
        } else {
          l_run += (gv[0] + gv[1]) + (gv[2] + gv[3]);
        }
      }
      if constexpr (INTER) {  // an empty statement that "uses" the results keeps the piece in its round
        if constexpr (ONLINE) asm volatile("" : "+v"(sv), "+v"(tt), "+v"(gv), "+v"(tmx), "+v"(l_run), "+v"(m_run), "+v"(f_pub));
        else asm volatile("" : "+v"(sv), "+v"(tt), "+v"(gv));
      }
    };
    auto after_round = [&](auto i_tag) __attribute__((always_inline)) {
      if constexpr (INTER) {
        constexpr int i = decltype(i_tag)::value;
        static_for<NP>([&](auto k_tag) __attribute__((always_inline)) {
          if constexpr (decltype(k_tag)::value * MC / NP == i) piece(k_tag);
        });
        __builtin_amdgcn_sched_barrier(0);  // the rounds stay in order
      }
    };
    const unsigned so3 = (so2 + C::STAGE >= RING) ? so2 + C::STAGE - RING : so2 + C::STAGE;   // tile u+3
    if (gw) phase2(gf, wave_tag, t_pf, so4, so3, after_round);
    if (xw) {
      if constexpr (!INTER) static_for<NP>(piece);
      if constexpr (ONLINE) {
        need_pub = __builtin_amdgcn_ballot_w64(need) != 0 ? 1 : 0;
        if (ga.on_argmax) {
#pragma unroll
          for (int e = 0; e < 4; e++) {   // increasing j: a strict > keeps the smallest index
            const bool gt = tt[e] > best_v;
            best_v = gt ? tt[e] : best_v;
            best_i = gt ? b0 + e : best_i;
          }
        }
        if ((unsigned)(r_a - b0) < 4u) {
          // the positive: seen by exactly one lane of one split.  Its own term (p_{i r_i} - 1) p_{r_i} is formed in
          // fp32 by the kernel that finishes dQ: left in the bf16 sum it would cancel against - p_{r_i} with the
          // rounding error of a coefficient near 1
          // (rows past the end of this split belong to the next one; a positive that the self-mask removes keeps
          // its -inf, so that row's loss is +inf)
          if (a_q < No && r_a < send) ga.on_pos[a_q] = tt[r_a - b0];
#pragma unroll
          for (int e = 0; e < 4; e++)
            if (r_a - b0 == e) gv[e] = 0.f;
        }
        gq = __builtin_convertvector(gv, bf16x4);
      } else {
        // the rest touches few tiles and is decided per wave: 0 at the positive (j == r_i; its term is added in fp32
        // by the kernel that sums the partials, see PosFix), zeros for rows past the end of the split and on the
        // diagonal (i == j)
        bool hit_any;
        if (OWNER_IS_Q) hit_any = (unsigned)(r_a - b0) < 4u;
        else hit_any = (pos_r[0] == a_q) | (pos_r[1] == a_q) | (pos_r[2] == a_q) | (pos_r[3] == a_q);
        const int t1 = b0 - 4 * g16;
        const bool tail = !STEADY && (t1 + GR_T > send);
        const bool diag = ga.mask_self && (t1 < a0 + GR_OWN) && (t1 + GR_T > a0);
        if (__builtin_amdgcn_ballot_w64(hit_any) != 0 || tail || diag) {
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const bool hit = OWNER_IS_Q ? (r_a - b0 == e) : (pos_r[e] == a_q);
            if (hit || b0 + e >= send || (ga.mask_self && b0 + e == a_q)) gv[e] = 0.f;
          }
        }
        gq = __builtin_convertvector(gv, bf16x4);
      }
    }
    // the iteration after this one may be a steady one, which expects the phase-1 fragments of its tile (u+3) in
    // registers
    if (!STEADY && u + 3 < nt) {
      wait_vmem<0>();
      p1_load(so3, 0, C::KS);
    }
    if (!STEADY && pf) prefetch(u + 4, so4);  // in a steady iteration phase 2 has issued these loads
  };
  // ---- prologue: start the first tiles, phase 1 of tile 0 ------------------------------------------------------
#pragma unroll 1
  for (int u = 0; u < min(nt, 4); u++) prefetch(u, u * C::STAGE);
  wait_vmem<0>();
  // (the compiler's own loads end here: a wait of its own for these two inside the loop would be for the loads into LDS as well)
  if constexpr (SYM) asm volatile("" : "+v"(lse_a), "+v"(r_a));
  p1_load(0, 0, C::KS);
  p1_mfma(0, C::KS);
  auto next_stage = [&](unsigned so) __attribute__((always_inline)) -> unsigned { return (so + C::STAGE >= RING) ? so + C::STAGE - RING : so + C::STAGE; };
  unsigned so = RING - C::STAGE;  // stage of "tile -1"
  constexpr std::integral_constant<int, -1> unsteady{};
  constexpr std::integral_constant<int, -1> any_stage{};
  body(-1, so, any_stage, unsteady);
  so = 0;
  int u = 0;
  auto steady_loop = [&](auto wave_tag) __attribute__((always_inline)) {
    if constexpr (D == 768) {
      // the widest kernel (the headline shape) is unrolled over the ring: five iterations per trip, tile u is in
      // stage u % 5 and u is a multiple of 5 here (so stays 0); measured 4 % on the dP walk.  The other widths keep
      // the rolled loop (five copies of every width would more than double the time this file takes to compile).
#pragma unroll 1
      for (; u + GR_STAGES + 4 < nt; u += GR_STAGES) {
        static_for<GR_STAGES>([&](auto stage_tag) __attribute__((always_inline)) {
          body(u + decltype(stage_tag)::value, 0u, stage_tag, wave_tag);
        });
      }
    } else {
#pragma unroll 1
      for (; u + 5 < nt; u++) { body(u, so, any_stage, wave_tag); so = next_stage(so); }
    }
  };
  // (the steady body of the one-direction kernels has no place for the diagonal mask: with mask_self every
  // iteration takes the general body)
  if (SYM || !ga.mask_self) {
    switch (__builtin_amdgcn_readfirstlane(w)) {
      case 0: steady_loop(std::integral_constant<int, 0>{}); break;
      case 1: steady_loop(std::integral_constant<int, 1>{}); break;
      case 2: steady_loop(std::integral_constant<int, 2>{}); break;
      default: steady_loop(std::integral_constant<int, 3>{}); break;
    }
  }
#pragma unroll 1
  for (; u < nt; u++) { body(u, so, any_stage, unsteady); so = next_stage(so); }

  // ---- epilogue: scale by alpha / B and store the owned rows ---------------------------------------------------------
  float* out = OWNER_IS_Q ? (ga.dq_out + (size_t)split * ga.dq_split_stride) : (ga.dp_out + (size_t)split * ga.dp_split_stride);
#pragma unroll
  for (int mt = 0; mt < 2; mt++)
#pragma unroll
    for (int ct = 0; ct < C::CT; ct++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int a = a0 + 32 * mt + 8 * (r >> 2) + 4 * h + (r & 3);
        if (a < No) out[(size_t)a * D + w * C::DS + 32 * ct + ln] = acc[mt][ct][r] * ga.out_scale;
      }
  if constexpr (ONLINE) {  // the row's statistics of this split
    const float l_sum = sum_g16(l_run);
    if (ga.on_argmax) argmax_g16(best_v, best_i);
    if (g16 == 0 && a_q < No) {
      // (reference, sum 2^(t - reference)) is all the log-sum-exp needs: the same bits whether or not the
      // arg-max is tracked
      const size_t o = (size_t)split * No + a_q;
      ga.on_ref[o] = m_run;
      ga.on_l[o] = l_sum;
      if (ga.on_argmax) { ga.on_best[o] = best_v; ga.on_idx[o] = best_i; }
    }
  }
}

}  // namespace gc
