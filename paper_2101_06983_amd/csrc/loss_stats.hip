// Statistics pass of the bf16 loss path for gfx950 (widths from 256; d = 128: loss_mfma128.hip), Eq. 1 / Eq. 4: per anchor,
// online max and sum of 2^t over target tiles, the positive's score and the argmax; the score tile lives in MFMA
// accumulators only.
#include "mfma_common.h"
#include "stats_tile.h"

namespace gc {

// ===========================================================================
// Statistics pass.  Workgroup = 512 threads = 8 waves as 2 (targets, M) x 4 (anchors, N); wave tile MT x NT MFMA tiles.
// k is staged through LDS in chunks of 64, two stages.  2 x 1: workgroup tile 128 x 128, two workgroups to a compute unit.
// 4 x 2: 256 x 256, one workgroup to a compute unit, for the largest calls (see stats_block).
// ===========================================================================
constexpr int ST_KC = 64, ST_ROWB = ST_KC * 2;           // bytes per LDS row (8 chunks of 16 bytes, unpadded)
constexpr int stats_stage_bytes(int block) { return 2 * block * ST_ROWB; }   // one stage: the target rows, then the anchor rows
// LDS layout: chunk c of row r is stored at chunk position c ^ ((r >> 1) & 7): the 16 rows that a
// 16-lane group reads in one fragment load then fall into 16 different 16-byte bank groups.

// ARGMAX: the plain pass with the first index of the maximum; BOTH, TRI: the statistics of both sides of the symmetric forms
// from one pass over the scores (see kBothMin), TRI (NT-Xent, q = p) over the tiles on and above the diagonal only.
enum StatsMode { ST_PLAIN, ST_ARGMAX, ST_BOTH, ST_TRI };
template <StatsMode MODE, int BLOCK>
__global__ void __launch_bounds__(512, BLOCK == kStatBlock ? 4 : 2) stats_mfma_kernel(StatsArgs g) {
  constexpr int MT = BLOCK / 64, NT = BLOCK / 128, ST_TM = BLOCK, ST_TN = BLOCK;
  constexpr int ST_STAGE_BYTES = stats_stage_bytes(BLOCK);
  constexpr int LROWS = ST_TM / 4;   // rows of a stage that a wave loads
  constexpr bool TRI = MODE == ST_TRI, BOTH = MODE == ST_BOTH || TRI, ARGMAX = MODE == ST_ARGMAX;
  const unsigned short* const Q = g.Q;
  const unsigned short* const Pm = g.P;
  const int32_t* const pos_idx = g.pos_idx;
  const int B = g.B, P = g.Pn, d = g.d, cols_per_split = g.cols_per_split;
  const float alpha2 = g.alpha2;
  const int mask_self = BOTH ? 0 : g.mask_self;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_b[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  if constexpr (BOTH) both_begin(g);
  int task = xcd_task_id(), ablk, split;
  if (TRI) split = tri_task(task, P, ST_TN, cols_per_split, ablk);
  else { ablk = task % g.n_ablk; split = task / g.n_ablk; }
  const int a0 = ablk * ST_TN;
  const int cbeg = (TRI ? a0 : 0) + split * cols_per_split, cend = min(P, cbeg + cols_per_split);
  const int nk = d / ST_KC;

  // ---- direct global->LDS loads: wave w fills rows LROWS w .. of a stage (waves 0-3 the target rows,
  // waves 4-7 the anchor rows), each instruction 8 rows x 8 chunks ------------------------------------
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);  // as a scalar: what follows from it stays uniform
  const bool loads_q = wave_u >= 4;
  const unsigned short* lmat = loads_q ? Q : Pm;
  const int lrows = loads_q ? B : P;
  const int lrow_in = (wave_u & 3) * LROWS + (lane >> 3);  // + 8 j: row inside the tile
  const unsigned stage_m0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)smem_b + wave_u * LROWS * ST_ROWB);
  auto src_of = [&](int j, int tile_row0, bool clamp) -> unsigned {  // byte offset from the tile's first row, chunk kc = 0
    int r = lrow_in + 8 * j;
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    if (clamp) r = min(r, lrows - 1 - tile_row0);
    return (unsigned)(r * d * 2 + c * 16);
  };
  // full tile: row 8 j moves the chunk by its swizzle's bit 2 only, so two offsets and a scalar step serve all loads
  const unsigned voff_full[2] = {src_of(0, 0, false), src_of(1, 0, false) - 16u * (unsigned)d};
  auto prefetch = [&](int tile_row0, int kc, int stage) __attribute__((always_inline)) {
    const unsigned short* base_v = lmat + (size_t)tile_row0 * d + kc * ST_KC;  // the same in every lane of a wave
    const unsigned long long bu = (unsigned long long)(uintptr_t)base_v;
    const unsigned short* base = (const unsigned short*)(uintptr_t)(
        // readfirstlane returns int: go through unsigned, or the low half sign-extends into the high one
        ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)(bu >> 32)) << 32) |
        (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)bu));
    const unsigned m0 = stage_m0 + stage * ST_STAGE_BYTES;
    if (tile_row0 + ST_TM <= lrows) {
#pragma unroll
      for (int j = 0; j < LROWS / 8; j++) dma_group<1>((const char*)base + 16 * j * d, &voff_full[j & 1], m0 + 1024 * j);
    } else {  // ragged tile: rows past the end re-read the last valid row (masked later)
#pragma unroll
      for (int j = 0; j < LROWS / 8; j++) {
        const unsigned off = src_of(j, tile_row0, true);
        dma_group<1>(base, &off, m0 + j * 1024);
      }
    }
  };

  // ---- fragment addresses: row (lane & 31) of an MFMA tile, chunk 2 ks + (lane >> 5), swizzled ---------
  const int swz_l = ((lane & 31) >> 1) & 7;
  unsigned koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ks++) koff[ks] = (unsigned)(((2 * ks + (lane >> 5)) ^ swz_l) * 16);
  const unsigned char* a_base = smem_b + (wm * 32 * MT + (lane & 31)) * ST_ROWB;               // + mt * 32 rows
  const unsigned char* b_base = smem_b + (ST_TM + wn * 32 * NT + (lane & 31)) * ST_ROWB;        // + nt * 32 rows

  // per-lane running statistics for its anchor columns
  float rm[NT], rl[NT], rpos[NT];
  int ridx[NT], a_col[NT], r_of[NT];
#pragma unroll
  for (int nt = 0; nt < NT; nt++) {
    rm[nt] = -INFINITY; rl[nt] = 0.f; rpos[nt] = 0.f; ridx[nt] = 0x7fffffff;
    a_col[nt] = a0 + wn * 32 * NT + nt * 32 + (lane & 31);
    r_of[nt] = (a_col[nt] >= B) ? -1 : TRI ? a_col[nt] ^ 1 : pos_idx[a_col[nt]];
  }
  // BOTH: sums with the reference 0 (rm, rl: of the tiles that needed one of their own); whether this lane saw the positive
  float lf[NT];
  bool got[NT];
#pragma unroll
  for (int nt = 0; nt < NT; nt++) { lf[nt] = 0.f; got[nt] = false; }
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  f32x2* cbuf = (f32x2*)(smem_b + 2 * ST_STAGE_BYTES);   // [4 wn][ST_TM columns] (maximum, sum)
  const int col_in = 8 * (reduce16_reg_of(lane) >> 2) + 4 * (lane >> 5) + (reduce16_reg_of(lane) & 3);
  const bool own_edge = a0 + wn * 32 * NT + 32 * NT > B;
  bool fast = true;   // (of this wave) the sums of the last tile that took references of its own were within the bounds

  // The k-chunks of all the tiles of this workgroup form one sequence of steps; step st lives in stage st & 1 and
  // its loads are issued one step ahead inside a tile.  (Loading the first chunk of the next tile under the last
  // MFMAs of this one was measured too: no gain at 2 tiles of 12 chunks, a loss at 16 tiles of 2 chunks.)
  int st = 0;
  for (int b0 = cbeg; b0 < cend; b0 += ST_TM) {
    f32x16 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
      for (int nt = 0; nt < NT; nt++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[mt][nt][r] = 0.f;

    const int row0 = loads_q ? a0 : b0;
    // nothing is in flight and every reader is past the last barrier: both stages are free
    prefetch(row0, 0, st & 1);
    wait_vmem<0>();
    lds_barrier();
    bf16x8 af[2][MT], bfg[2][NT];
    for (int kc = 0; kc < nk; kc++, st++) {
      if (kc + 1 < nk) prefetch(row0, kc + 1, (st + 1) & 1);
      const int so = (st & 1) * ST_STAGE_BYTES;
      __builtin_amdgcn_iglp_opt(0);  // scheduler hint: interleave the fragment reads with the MFMA stream
      auto load_frags = [&](int ks, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MT; mt++) af[buf][mt] = *(const bf16x8*)(a_base + so + mt * 32 * ST_ROWB + koff[ks]);
#pragma unroll
        for (int nt = 0; nt < NT; nt++) bfg[buf][nt] = *(const bf16x8*)(b_base + so + nt * 32 * ST_ROWB + koff[ks]);
      };
      load_frags(0, 0);
#pragma unroll
      for (int ks = 0; ks < ST_KC / 16; ks++) {
        if (ks + 1 < ST_KC / 16) load_frags(ks + 1, (ks + 1) & 1);
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
          for (int nt = 0; nt < NT; nt++) acc[mt][nt] = mfma32(af[ks & 1][mt], bfg[ks & 1][nt], acc[mt][nt]);
      }
      wait_vmem<0>();   // this wave's part of the next stage has landed
      lds_barrier();  // ... and everybody's; nobody still reads the stage that is overwritten next
    }

    // ---- tile epilogue: online softmax statistics, all in registers; acc holds the raw dot products, the
    // base-2 logit is t = alpha2 * acc (alpha2 > 0: the order of the raw values is the order of the logits) -------
    const int brow0 = b0 + wm * 32 * MT + 4 * (lane >> 5);  // + mt*32 + 8*(r/4) + r%4
    const bool edge = (b0 + ST_TM > cend);
    if constexpr (BOTH) {
      bool has_pos = false;
#pragma unroll
      for (int nt = 0; nt < NT; nt++) has_pos = has_pos || (unsigned)(r_of[nt] - b0) < (unsigned)ST_TM;
      if (__builtin_amdgcn_ballot_w64(has_pos) != 0) {
#pragma unroll
        for (int nt = 0; nt < NT; nt++)
#pragma unroll
          for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int r = 0; r < 16; r++)
              if (brow0 + mt * 32 + 8 * (r >> 2) + (r & 3) == r_of[nt] && r_of[nt] < cend) {
                rpos[nt] = acc[mt][nt][r] * alpha2; got[nt] = true;
                acc[mt][nt][r] = -INFINITY;   // the positive is no part of the sums (both_merge_kernel adds it)
              }
      }
      const bool cols = !TRI || b0 > a0;
      const bool masked = edge || own_edge || (TRI && !cols);
      bool done = false;
      if (!masked && fast) {
        float rs[NT], c[MT], lo = INFINITY, hi = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; nt++) rs[nt] = 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
          float v[16];
#pragma unroll
          for (int r = 0; r < 16; r++) {
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
              const float e = fast_exp2(acc[mt][nt][r] * alpha2);
              rs[nt] += e;
              v[r] = nt ? v[r] + e : e;
            }
          }
          c[mt] = reduce16_lanes32<false>(v, lane);
          lo = fminf(lo, c[mt]); hi = fmaxf(hi, c[mt]);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int nt = 0; nt < NT; nt++) { lo = fminf(lo, rs[nt]); hi = fmaxf(hi, rs[nt]); }
        if (__builtin_amdgcn_ballot_w64(!(lo >= kBothMin && hi <= kBothMax)) == 0) {
#pragma unroll
          for (int nt = 0; nt < NT; nt++) lf[nt] += rs[nt];
          if (!(lane & 1)) {
#pragma unroll
            for (int mt = 0; mt < MT; mt++) cbuf[wn * ST_TM + wm * 32 * MT + mt * 32 + col_in] = f32x2{0.f, c[mt]};
          }
          done = true;
        }
      }
      if (!done) {   // masks, and references of its own for every row and column
        if (masked) {
#pragma unroll
          for (int nt = 0; nt < NT; nt++)
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
              for (int r = 0; r < 16; r++) {
                const int j = brow0 + mt * 32 + 8 * (r >> 2) + (r & 3);
                if (j >= cend || a_col[nt] >= B || (TRI && j == a_col[nt])) acc[mt][nt][r] = -INFINITY;
              }
        }
        float lo = INFINITY, hi = -INFINITY;   // of the references
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
          float tm = -INFINITY, sum = 0.f;
#pragma unroll
          for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int r = 0; r < 16; r++) tm = fmaxf(tm, acc[mt][nt][r]);
          tm *= alpha2;
          lo = fminf(lo, tm); hi = fmaxf(hi, tm);
          if (tm == -INFINITY) continue;
          const float mn = fmaxf(rm[nt], tm);
#pragma unroll
          for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int r = 0; r < 16; r++) sum += fast_exp2(__builtin_fmaf(acc[mt][nt][r], alpha2, -mn));
          rl[nt] = rl[nt] * fast_exp2(rm[nt] - mn) + sum;
          rm[nt] = mn;
        }
        if (cols) {
#pragma unroll
          for (int mt = 0; mt < MT; mt++) {
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; r++) {
              v[r] = acc[mt][0][r];
#pragma unroll
              for (int nt = 1; nt < NT; nt++) v[r] = fmaxf(v[r], acc[mt][nt][r]);
            }
            const float cm = reduce16_lanes32<true>(v, lane) * alpha2, cs = cm == -INFINITY ? 0.f : cm;
            static_for<16>([&](auto r_tag) __attribute__((always_inline)) {
              constexpr int r = decltype(r_tag)::value;
              const float m = reduce16_spread<r>(cs);
#pragma unroll
              for (int nt = 0; nt < NT; nt++) v[r] = (nt ? v[r] : 0.f) + fast_exp2(__builtin_fmaf(acc[mt][nt][r], alpha2, -m));
            });
            const float cl = reduce16_lanes32<false>(v, lane);
            lo = fminf(lo, cm); hi = fmaxf(hi, cm);
            if (!(lane & 1)) cbuf[wn * ST_TM + wm * 32 * MT + mt * 32 + col_in] = f32x2{cm, cl};
            __builtin_amdgcn_sched_barrier(0);
          }
          // (a sum relative to its maximum is in 1 .. 32)
          if (!masked) fast = __builtin_amdgcn_ballot_w64(!(lo >= kBothMinLog2 && hi <= kBothMaxLog2 - 5)) == 0;
        }
      }
      if (cols) {   // the four waves' sums of a column, in wave order (the next tile writes them behind many barriers)
        lds_barrier();
        if (tid < ST_TM && b0 + tid < cend) {
          f32x2 x[4];
          float m = -INFINITY, l = 0.f;
#pragma unroll
          for (int k = 0; k < 4; k++) { x[k] = cbuf[k * ST_TM + tid]; m = fmaxf(m, x[k][0]); }
          const float ms = m == -INFINITY ? 0.f : m;
#pragma unroll
          for (int k = 0; k < 4; k++) l += x[k][1] * fast_exp2(x[k][0] - ms);
          const size_t o = (size_t)ablk * P + b0 + tid;
          g.col_m[o] = m; g.col_l[o] = l;
        }
      }
      continue;
    }
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      const int a = a_col[nt];
      // the masks that can touch this tile
      const bool diag = mask_self && (a >= b0 && a < b0 + ST_TM);
      const bool haspos = (unsigned)(r_of[nt] - b0) < (unsigned)ST_TM;
      if (edge || diag || haspos) {  // rare: the general slow walk
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
          for (int r = 0; r < 16; r++) {
            int j = brow0 + mt * 32 + 8 * (r >> 2) + (r & 3);
            if (j == r_of[nt]) rpos[nt] = acc[mt][nt][r] * alpha2;
            if (j >= cend || (mask_self && j == a)) acc[mt][nt][r] = -INFINITY;
          }
      }
      // tile max + first index attaining it (rows are visited in increasing j within mt; across
      // register order j is increasing too, so a strict > keeps the smallest index)
      float tmr = -INFINITY; int tc = 0;
#pragma unroll
      for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const float t = acc[mt][nt][r];
          if constexpr (ARGMAX) {
            const bool le = t <= tmr;
            tmr = le ? tmr : t;
            tc = le ? tc : (mt * 32 + 8 * (r >> 2) + (r & 3));
          } else {
            tmr = fmaxf(tmr, t);
          }
        }
      if (tmr > -INFINITY) {
        const float tm = tmr * alpha2;
        const float mn = fmaxf(rm[nt], tm);
        float s = 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
          for (int r = 0; r < 16; r++) s += fast_exp2(__builtin_fmaf(acc[mt][nt][r], alpha2, -mn));
        rl[nt] = rl[nt] * fast_exp2(rm[nt] - mn) + s;
        if (ARGMAX && tm > rm[nt]) ridx[nt] = brow0 + tc;  // later tiles have larger j: strict >
        rm[nt] = mn;
      }
    }
  }

  // ---- combine the two half-waves (same anchor column, different target rows) -------------------
#pragma unroll
  for (int nt = 0; nt < NT; nt++) {
    if constexpr (BOTH) stat_merge(rm[nt], rl[nt], ridx[nt], lf[nt] > 0.f ? 0.f : -INFINITY, lf[nt], 0x7fffffff);
    float m2 = __shfl_xor(rm[nt], 32), l2 = __shfl_xor(rl[nt], 32);
    int i2 = __shfl_xor(ridx[nt], 32);
    stat_merge(rm[nt], rl[nt], ridx[nt], m2, l2, i2);
  }
  // ---- combine the two waves along M through LDS, then write the split partial ------------------
  __syncthreads();
  float* xs = (float*)smem_b;  // [4 wn][NT][32][3]
  if (wm == 1 && lane < 32) {
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      float* x = xs + ((wn * NT + nt) * 32 + lane) * 3;
      x[0] = rm[nt]; x[1] = rl[nt]; x[2] = __builtin_bit_cast(float, ridx[nt]);
    }
  }
  __syncthreads();
  if (wm == 0 && lane < 32) {
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      const float* x = xs + ((wn * NT + nt) * 32 + lane) * 3;
      stat_merge(rm[nt], rl[nt], ridx[nt], x[0], x[1], __builtin_bit_cast(int, x[2]));
      int a = a_col[nt];
      if (a < B) {
        g.row_m[(size_t)split * B + a] = rm[nt];
        g.row_l[(size_t)split * B + a] = rl[nt];
        if constexpr (ARGMAX) g.row_idx[(size_t)split * B + a] = ridx[nt];
      }
    }
  }
  // the positive's score is seen by exactly one lane of one workgroup
#pragma unroll
  for (int nt = 0; nt < NT; nt++) {
    int a = a_col[nt], r = r_of[nt];
    if constexpr (BOTH) {
      if (got[nt] && a < B) g.pos_t[a] = rpos[nt];
      continue;
    }
    if (a < B && r >= cbeg && r < cend) {
      // lane that held row r: rows of this lane are brow(mt, reg) with 4*(lane>>5) offset
      int rel = (r - cbeg) % ST_TM;  // row inside its tile
      int wmr = rel / (32 * MT), in = rel % (32 * MT);
      int half = (in % 8) / 4;
      // a positive that the self-mask removes has the logit -inf (its row loss is then +inf)
      if (wmr == wm && half == (lane >> 5)) g.pos_t[a] = (mask_self && r == a) ? -INFINITY : rpos[nt];
    }
  }
}

// ===========================================================================
// Statistics pass for few scores: 32 x 32 tiles, the contraction split over the four waves of a workgroup in 64-wide
// chunks, every operand loaded straight into registers (lane (n, h) takes elements 32 h .. 32 h + 31 of a chunk of its
// row, so that two lanes use a whole 128-byte line; any order of k works if both operands share it).  Tiles staged through
// LDS are all latency of dependent k-chunks at these sizes; here a wave has all its loads in flight at once: 6.6 us at
// 128 x 256 x 768.  It costs B P d / 8 bytes of L2 traffic, so that the staged tiles (128 x 128; d = 128: 256 anchors) win again.
//   loss alone, us (32 x 32 / staged)   2^18 scores   2^19          2^20          2^21
//     d = 128                           12.3 / 26.0   14.7 / 26.1   15.3 / 26.3   22.0 / 26.8
//     d = 256                           13.6 / 14.3   14.8 / 14.3   16.9 / 14.4   23.6 / 14.4
//     d = 512                           13.7 / 15.2   17.0 / 15.5   19.4 / 15.0   29.6 / 16.1
//     d = 768                           14.3 / 16.6   19.0 / 16.9   22.4 / 16.9   37.0 / 17.3
// The line, 2^20, is that of the gradient kernel for few scores, which merges these statistics (a call with it instead of a merge
// and the long walks: 1 to 14 % shorter at 2^20); between 2^18.5 and 2^20 the statistics alone would be 0.5 to 5 us shorter with staged tiles.
// ===========================================================================
__global__ void __launch_bounds__(256) stats_small_kernel(StatsSmallArgs g) {
  constexpr int T = kStatTile, PD = 3;
  __shared__ StatTileLds lds;
  if (g.inv) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i == 0) *g.shared = 0;
    if (i < g.B) {   // (at least one workgroup of 256 threads per 32 anchors)
      const int r = g.pos_idx[i];
      if (r >= 0 && r < g.Pn) g.inv[r] = i;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, ln = lane & 31;
  const int task = xcd_task_id();
  const int a0 = (task % g.n_ablk) * T, split = task / g.n_ablk;
  const int nch = g.d / 64;
  const char* qp = (const char*)(g.Q + (size_t)min(a0 + ln, g.B - 1) * g.d + 32 * h);
  StatTile<false> st(g, a0);
  const int t_end = min(g.tiles, (split + 1) * g.tiles_per_split);
  for (int t = split * g.tiles_per_split; t < t_end; t++) {
    const int j0 = t * T;
    const char* pp = (const char*)(g.P + (size_t)min(j0 + ln, g.Pn - 1) * g.d + 32 * h);
    u32x4 fq[PD][4], fp[PD][4];
    auto issue = [&](int slot, int c) __attribute__((always_inline)) {
#pragma unroll
      for (int v = 0; v < 4; v++) {
        fq[slot][v] = *(const u32x4*)(qp + (size_t)c * 128 + 16 * v);
        fp[slot][v] = *(const u32x4*)(pp + (size_t)c * 128 + 16 * v);
      }
    };
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.f;
#pragma unroll
    for (int p = 0; p < PD; p++)
      if (wave + 4 * p < nch) issue(p, wave + 4 * p);
    for (int base = wave; base < nch; base += 4 * PD) {
#pragma unroll
      for (int p = 0; p < PD; p++) {
        const int c = base + 4 * p;
        if (c < nch) {
#pragma unroll
          for (int v = 0; v < 4; v++) acc = mfma32(__builtin_bit_cast(bf16x8, fp[p][v]), __builtin_bit_cast(bf16x8, fq[p][v]), acc);
          if (c + 4 * PD < nch) issue(p, c + 4 * PD);
        }
      }
    }
    StatTile<false>::put(lds, wave, acc);
    __syncthreads();
    st.tile(g, lds, j0);
    __syncthreads();   // the partial tiles have been read
  }
  st.finish(g, lds, split);
}
static hipError_t launch_stats_small(const LossArgs& a, const LossPlan& pl) {
  StatsSmallArgs g = stats_small_args(a, pl, (const unsigned short*)a.q, (const unsigned short*)a.p);
  if (merges_itself(a, pl)) { g.inv = (int32_t*)(a.ws + pl.off_inv); g.shared = (int*)(a.ws + pl.off_err) + 1; }
  stats_small_kernel<<<g.n_ablk * pl.stat_splits, 256, 0, a.stream>>>(g);
  return hipGetLastError();
}

// Rows and columns of a workgroup's scores.  128 fills the chip from few scores on (1021 x 4099 x 384: 68 blocks of 256 leave
// most of it idle, 27.6 us for the loss alone, 17.0 so) and is as fast or faster almost everywhere, in spite of twice the LDS bytes per MFMA:
//   loss alone, us (256 / 128)   2^25 scores      2^26            2^28            2^29
//     d = 256                    40.1 / 33.3   70.1 / 57.2     231 / 186       428 / 354
//     d = 512                    53.1 / 48.9   99.4 / 92.5     333 / 324       627 / 625
//     d = 640                    59.6 / 56.6    113 / 111      381 / 391       725 / 773
//     d = 768                    65.6 / 66.2  121..127 / 129   431 / 470       815 / 917
// but reads the inputs twice as often, past what an XCD's L2 holds of wide rows: at 2^27 scores 199 / 203 (d = 640), 227 / 239 (768);
// at 6000 x 12000 x 768, 2^26.1, whose last blocks of 256 are part empty, 145 / 139.
int stats_block(int B, int P, int d) { return d >= 640 && (long long)B * P >= (1ll << 27) ? 256 : kStatBlock; }

template <StatsMode MODE, int BLOCK>
static hipError_t stats_mfma_launch_as(const StatsArgs& g, int nwg, hipStream_t stream) {
  constexpr int smem = 2 * stats_stage_bytes(BLOCK) + (MODE >= ST_BOTH ? 4 * BLOCK * 8 : 0);
  static bool attr_done[64];
  if (hipError_t e = ensure_dyn_lds((const void*)stats_mfma_kernel<MODE, BLOCK>, smem, attr_done); e != hipSuccess) return e;
  stats_mfma_kernel<MODE, BLOCK><<<nwg, 512, smem, stream>>>(g);
  return hipGetLastError();
}
template <StatsMode MODE>
static hipError_t stats_mfma_launch(const StatsArgs& g, int block, int splits, hipStream_t stream) {
  return block == 256 ? stats_mfma_launch_as<MODE, 256>(g, g.n_ablk * splits, stream) : stats_mfma_launch_as<MODE, kStatBlock>(g, g.n_ablk * splits, stream);
}
hipError_t launch_stats_mfma(const LossArgs& a, const LossPlan& pl) {
  if (pl.stat_tile) return launch_stats_small(a, pl);
  if (a.d == 128) return launch_stats128(a, pl);   // whole anchor rows in registers: a kernel of its own
  char* ws = a.ws;
  StatsArgs g{};
  g.Q = (const unsigned short*)a.q; g.P = (const unsigned short*)a.p; g.pos_idx = a.pos_idx; g.B = a.B; g.Pn = a.P; g.d = a.d;
  g.alpha2 = a.alpha * kLog2e; g.mask_self = (a.flags & GC_MASK_SELF) ? 1 : 0;
  const int block = stats_block(a.B, a.P, a.d);
  g.n_ablk = (a.B + block - 1) / block; g.cols_per_split = pl.stat_cols_per_split;
  g.row_m = (float*)(ws + pl.off_part_m); g.row_l = (float*)(ws + pl.off_part_l); g.row_idx = (int*)(ws + pl.off_part_idx);
  g.pos_t = (float*)(ws + pl.off_pos);
  return a.argmax ? stats_mfma_launch<ST_ARGMAX>(g, block, pl.stat_splits, a.stream) : stats_mfma_launch<ST_PLAIN>(g, block, pl.stat_splits, a.stream);
}

// ---- statistics of both sides (the symmetric forms) ------------------------------------------------------------------
// One pass where the plain one does not have its tiles for few scores.  At most 128 blocks: each leaves a partial per column
// (n^2 / 16 bytes), and they lie where the gradient pass will put its own: where that has few splits, and so little room, the
// plain passes stay as well (`use`; 32768 x 128 for NT-Xent, 16384 x 256 for the symmetric loss).
BothPlan plan_both(int n, int d, bool triangle, const LossPlan& pl) {
  BothPlan b{};
  const int T = d == 128 ? 256 : kStatBlock, n_ablk = (n + T - 1) / T;
  if (pl.route != ROUTE_MFMA || pl.stat_tile || n_ablk > 128) return b;
  b.triangle = triangle;
  b.block = T;
  b.n_ablk = n_ablk;
  if (triangle) {
    // ranges of equal length (whole tiles: 32 rows at d = 128) that fill the chip once: the shortest, from the least that can be
    // (`rows`: of all blocks' walks, n - T k each.  Every call asks: 32 us of host time at 28000 x 128 with every length tried, 8.7 so)
    const int unit = d == 128 ? 32 : T, cap = 2 * num_cu();
    const long long rows = (long long)n * n_ablk - (long long)T * n_ablk * (n_ablk - 1) / 2;
    int len = (int)(rows / cap) / unit * unit;
    for (len = len < (d == 128 ? 64 : T) ? (d == 128 ? 64 : T) : len;; len += unit) {
      int wgs = 0;
      for (int k = 0; k < n_ablk; k++) wgs += (n - T * k + len - 1) / len;
      if (wgs > cap && len < n) continue;
      b.cols_per_split = len; b.nwg = wgs; b.row_slots = (n + len - 1) / len;
      break;
    }
  } else {
    b.cols_per_split = pl.stat_cols_per_split; b.row_slots = pl.stat_splits; b.nwg = n_ablk * pl.stat_splits;
  }
  b.use = (size_t)(b.row_slots + n_ablk) * n * 8 <= pl.off_dp_part - pl.off_dq_part;
  return b;
}
hipError_t launch_stats_both(const LossArgs& a, const LossPlan& pl, const BothPlan& b) {
  StatsArgs g{};
  g.Q = (const unsigned short*)a.q; g.P = (const unsigned short*)a.p; g.pos_idx = a.pos_idx; g.B = a.B; g.Pn = a.P; g.d = a.d;
  g.alpha2 = a.alpha * kLog2e; g.n_ablk = b.n_ablk; g.cols_per_split = b.cols_per_split;
  b.partials(a, pl, g.row_m, g.row_l, g.col_m, g.col_l);
  g.pos_t = (float*)(a.ws + pl.off_pos);
  g.zero = a.wide; g.inv = b.triangle ? nullptr : a.pos_inv;
  if (a.d == 128) return launch_stats128_both(g, b.triangle, b.nwg, a.stream);
  return b.triangle ? stats_mfma_launch_as<ST_TRI, kStatBlock>(g, b.nwg, a.stream) : stats_mfma_launch_as<ST_BOTH, kStatBlock>(g, b.nwg, a.stream);
}

}  // namespace gc
