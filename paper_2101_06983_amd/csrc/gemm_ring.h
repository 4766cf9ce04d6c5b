// The tiled products of the encoder (mlp.hip): D[M x N] = A B, both operands streamed through LDS by direct global->LDS loads.
//
// A workgroup of 512 threads owns a (64 MT) x (64 NT) tile of D.  Its eight waves are 2 (k) x 2 (m) x 2 (n): four of them cover
// the tile, 32 MT x 32 NT each, and two such groups take turns at the k-steps of 16 of every stage; their sums meet in LDS at
// the end.  What a wave reads from LDS per MFMA falls with the size of its own tile ((MT + NT) / (MT NT) KB: 1.5 for 32 x 64, 1 for
// 64 x 64, 0.83 for 64 x 96, where a compute unit delivers 1 KB in the 8 cycles that an MFMA of each of its four SIMDs leaves),
// and the loads into LDS with the workgroup's, so the tiles are as large as the registers allow with two waves per SIMD; splitting k
// and not the tile between the two costs neither.
//
// Operands reach LDS in stages of SUBS k-steps, a ring of NS of them; loads are issued NS - 1 stages ahead, one barrier a stage.
// Three layouts in memory, each written to LDS so that fragment reads are free of bank conflicts:
//   FragOp  fragments, 1 KB each: [k-step of 16][32-wide tile][plane], lane l holding index l % 32 and 8 of the 16 k
//   RowOp   rows with k contiguous, 128 bytes of each row a stage; 16-byte chunks XORed with bits of the row
//   ColOp   rows of k with the index contiguous (transposing reads): the weights as they are stored, too
// Measured at 1536 rows, 1024-3072-768 (us, with 64 x 128 tiles staged through registers in LDS before, the gradients by single
// waves that read fragments from L2): hidden layer 33.8 -> 21.0, second layer 27.0 -> 22.3, Act and dH 62.4 -> 38.5, parameter
// gradients 72.9 -> 46.4.  No unit is near full there (counters): the matrix pipe of a unit with a workgroup is busy 33, 40, 43 and 57 % of its
// time, LDS reads and writes take 17 to 21 %, without conflicts; waves wait a third of the time for loads or a barrier.  The start of a
// launch, GELU and the stores have no other workgroup of the unit to cover them: the more stages a workgroup has, the less they weigh.
// Within a k-step lane half h holds k 8 h .. 8 h + 7 ("plain") or {0..3, 8..11} + 4 h ("as an MFMA leaves it": register r of a
// result is row 8 (r / 4) + 4 h + r % 4); any order will do as long as both operands of a product share it.
#pragma once
#include "mfma_common.h"

namespace gc {

constexpr int RG_THREADS = 512, RG_WAVES = 8;

// piece p = wave + W i of a stage is 1 KB (W waves, eight but for mlp_grads_few_kernel); PIECES need not be a multiple of W: the
// last round is then not for all waves
template <int PIECES, int W>
constexpr int ring_rounds() { return (PIECES + W - 1) / W; }

// I32: 32-wide tiles of the index; P: planes; SUBS: k-steps a stage; X holds CT tiles a k-step
template <int I32, int P, int SUBS_, int W = RG_WAVES>
struct FragOp {
  static constexpr int SUBS = SUBS_, PIECES = I32 * P * SUBS, N = ring_rounds<PIECES, W>();
  const char* base; unsigned off[N]; size_t stage_bytes;
  __device__ __forceinline__ FragOp(const unsigned short* X, int CT, int tile0, int step0, int w) {
    base = (const char*)X + ((size_t)step0 * CT + tile0) * P * 1024;
    stage_bytes = (size_t)SUBS * CT * P * 1024;
    const int last = (CT - tile0) * P - 1;   // (tiles past the end repeat the last one; what they give is not stored)
#pragma unroll
    for (int i = 0; i < N; i++) {
      const int p = w + W * i;
      off[i] = (unsigned)((p / (I32 * P)) * CT * P + min(p % (I32 * P), last)) * 1024u;
    }
  }
  template <int I>
  __device__ __forceinline__ void load(int kt, unsigned lds, int w, int lane) const {
    dma_piece<0>(base + kt * stage_bytes + off[I], (unsigned)lane * 16u, lds + (unsigned)(w + W * I) * 1024u);
  }
  __device__ __forceinline__ static bf16x8 frag(const unsigned char* st, int sub, int t, int pl, int lane) {
    return *(const bf16x8*)(st + ((sub * I32 + t) * P + pl) * 1024 + lane * 16);
  }
};

// rows of one input or of two, the second from row first2 (a multiple of 32) on; rows past the end of either repeat its last one
struct RowSource {
  const void* x[2]; size_t ld;   // bytes
  int n1, n2, first2;
};
// 128 bytes of each row a stage: one plane of 64 values, or (P = 2) 32 high parts and 32 low parts
template <int ROWS, int P = 1>
struct RowOp {
  static constexpr int LINE = 128, SUBS = LINE / 32 / P, PIECES = ROWS * LINE / 1024, N = ring_rounds<PIECES, RG_WAVES>(), CH = LINE / 16;
  const char* base[N]; unsigned voff[N];
  __device__ __forceinline__ static int swz(int row) { return (row >> 1) & 7; }
  // row0: first row of the tile
  __device__ __forceinline__ RowOp(const RowSource& s, int row0, int w, int lane) {
#pragma unroll
    for (int i = 0; i < N; i++) {
      const int r = (w + RG_WAVES * i) * (64 / CH), dr = lane / CH;   // (a piece is 8 rows: never of both inputs)
      const bool second = s.n2 && row0 + r >= s.first2;
      const int local = second ? row0 + r - s.first2 : row0 + r, last = (second ? s.n2 : s.n1) - 1, first = min(local, last);
      base[i] = (const char*)s.x[second ? 1 : 0] + (size_t)first * s.ld;
      voff[i] = (unsigned)(min(local + dr, last) - first) * (unsigned)s.ld + (unsigned)(((lane % CH) ^ swz(r + dr)) * 16);
    }
  }
  template <int I>
  __device__ __forceinline__ void load(int kt, unsigned lds, int w, int) const {
    dma_piece<0>(base[I] + (size_t)kt * LINE, voff[I], lds + (unsigned)(w + RG_WAVES * I) * 1024u);
  }
  __device__ __forceinline__ static bf16x8 frag(const unsigned char* st, int sub, int t, int pl, int lane) {   // plain order
    const int ln = lane & 31, h = lane >> 5;
    const int c = 2 * sub + h + (P == 1 ? 0 : 4 * pl);
    return *(const bf16x8*)(st + (32 * t + ln) * LINE + ((c ^ swz(ln)) * 16));
  }
};

// 16 SUBS rows of k a stage, 32 I32 columns; two planes (P = 2): blocks of 32 high parts and 32 low parts along the columns, as RowOp.
// ORDER: of k within a step.  TAIL: k need not be a multiple of the stage; rows past the end repeat the last one, and ring_run makes
// the fragments of this operand zero there (the other operand's are finite or decide the result anyway).
enum ColOrder { COL_MFMA = 0, COL_PLAIN = 1 };
template <int I32, int P, int SUBS_, ColOrder ORDER, int W = RG_WAVES, bool TAIL_ = false>
struct ColOp {
  static constexpr bool TAIL = TAIL_;
  static constexpr int SUBS = SUBS_, LINE = I32 * P * 64, CH = LINE / 16, PIECES = 16 * SUBS * LINE / 1024, N = ring_rounds<PIECES, W>();
  // 64-byte quarters by the low bits of the row: the four rows that half a wave reads start 0 or 128 bytes apart (mod 256)
  __device__ __forceinline__ static int swz(int row) { return CH % 16 == 0 ? (row & 3) << 2 : ((row >> 1) & 1) << 2; }
  static_assert(CH % 8 == 0, "quarters change places within 128 bytes");
  const char* base; size_t ld; int rows, chunks, w0, lane0; unsigned voff[N];
  __device__ __forceinline__ unsigned source(int i, int last_row) const {
    const int q = (w0 + W * i) * 64 + lane0, row = q / CH, c = q % CH;
    return (unsigned)min(row, last_row) * (unsigned)ld + (unsigned)(min(c ^ swz(row), chunks - 1) * 16);
  }
  // ld: bytes; cols: of the matrix (tiles past the end repeat its last 16 bytes; what they give is not stored); rows: of k from row0 on
  __device__ __forceinline__ ColOp(const unsigned short* X, size_t ld_, int cols, int col0, int row0, int rows_, int w, int lane)
      : base((const char*)X + (size_t)row0 * ld_ + (size_t)col0 * 2 * P), ld(ld_), rows(rows_), chunks((cols - col0) * P / 8), w0(w), lane0(lane) {
#pragma unroll
    for (int i = 0; i < N; i++) voff[i] = source(i, 16 * SUBS - 1);
  }
  __device__ __forceinline__ int left(int kt) const { return rows - kt * 16 * SUBS; }   // rows of stage kt, if it is the last
  template <int I>
  __device__ __forceinline__ void load(int kt, unsigned lds, int w, int) const {
    unsigned v = voff[I];
    if (TAIL && left(kt) < 16 * SUBS) v = source(I, left(kt) - 1);
    dma_piece<0>(base + (size_t)kt * (16 * SUBS) * ld, v, lds + (unsigned)(w + W * I) * 1024u);
  }
  __device__ __forceinline__ static bf16x8 frag(const unsigned char* st, int sub, int t, int pl, int lane) {
    constexpr int PAIR = ORDER == COL_PLAIN ? 4 : 8;   // rows from the first four of a lane to the others (the same swz)
    const int h = lane >> 5, row = 16 * sub + (ORDER == COL_PLAIN ? 8 : 4) * h + ((lane & 15) >> 2);
    const int c = 4 * (P * t + pl) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    const unsigned char* p = st + row * LINE + ((c ^ swz(row)) * 16) + 8 * (lane & 1);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + PAIR * LINE));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
};
template <class A>
constexpr auto ring_tail(int) -> decltype(A::TAIL) { return A::TAIL; }
template <class A>
constexpr bool ring_tail(...) { return false; }

template <class A, class B>
constexpr int ring_stage_bytes() { return (A::PIECES + B::PIECES) * 1024; }

struct RingWave {
  int lane, w, kg, wm, wn;
  __device__ __forceinline__ RingWave() {
    lane = threadIdx.x & 63;
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    kg = w >> 2; wm = (w >> 1) & 1; wn = w & 1;
  }
};

template <int MT, int NT>
__device__ __forceinline__ void ring_zero(f32x16 (&acc)[MT][NT]) {
#pragma unroll
  for (int mt = 0; mt < MT; mt++)
#pragma unroll
    for (int nt = 0; nt < NT; nt++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[mt][nt][r] = 0.f;
}

// Piece round I (A's rounds, then B's) of the loads of stage kt, into the ring slot at LDS address `lds`
template <int I, class A, class B>
__device__ __forceinline__ void ring_issue(const A& a, const B& b, int kt, unsigned lds, const RingWave& wv) {
  if constexpr (I < A::N) {
    if ((I + 1) * RG_WAVES <= A::PIECES || wv.w + I * RG_WAVES < A::PIECES) a.template load<I>(kt, lds, wv.w, wv.lane);
  } else {
    constexpr int J = I - A::N;
    if ((J + 1) * RG_WAVES <= B::PIECES || wv.w + J * RG_WAVES < B::PIECES) b.template load<J>(kt, lds + A::PIECES * 1024, wv.w, wv.lane);
  }
}
__device__ __forceinline__ unsigned ring_lds(const unsigned char* smem) { return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)smem); }
// The rounds of a refill that run in the last k-step of a stage; the others run in the first of the next one, if the stages have two
template <class A, class B>
constexpr int ring_early() { return A::SUBS > 2 ? (A::N + B::N + 1) / 2 : A::N + B::N; }
// The first stages (LDS must be free), as far as ring_run expects them; what the wave does before ring_run hides their latency
template <int NS, class A, class B>
__device__ __forceinline__ void ring_fill(const A& a, const B& b, int nk, unsigned char* smem, const RingWave& wv) {
  const unsigned lds0 = ring_lds(smem);
#pragma unroll 1
  for (int s = 0; s < NS - 1 && s < nk; s++)
    static_for<A::N + B::N>([&](auto i) __attribute__((always_inline)) {
      ring_issue<decltype(i)::value>(a, b, s, lds0 + (unsigned)s * ring_stage_bytes<A, B>(), wv);
    });
  if (NS - 1 < nk)
    static_for<ring_early<A, B>()>([&](auto i) __attribute__((always_inline)) {
      ring_issue<decltype(i)::value>(a, b, NS - 1, lds0 + (unsigned)(NS - 1) * ring_stage_bytes<A, B>(), wv);
    });
}
// acc += this wave's share of the product over stages 0 .. nk - 1, after ring_fill.  PA, PB: planes; products of planes i and j
// with i + j < 2.  SMALL: those with i + j = 1 add up by themselves (beside acc each of them costs acc a rounding: for contractions so
// long that it shows).  Of a k-step the products of low parts come first where B has them, and last where A alone has:
// with them first there, every product is a little too small, which a sum over many rows shows (db1 of 65536 rows, 64-128-128: error
// 3.22e-6, of which -1.8e-6 in the mean; 2.67e-6 and -3.8e-7 so, 2.70e-6 and -4.1e-7 with products by one wave group).
// Ends behind a barrier: LDS is free.
// The fragments of the next k-step are read while the MFMAs of this one run, across the barrier of a stage too: it stands before the
// last k-step of the stage before.  Every wave then has the stage before in registers, whose slot takes the loads of the stage NS
// further on; they are spread over the MFMAs of that k-step and the next (a wave waits at a load until the unit's load path has
// taken it, one in 16 cycles: eight waves that issue theirs at once behind a barrier all wait for the last).
template <int MT, int NT, int PA, int PB, int NS, bool SMALL = false, class A, class B>
__device__ __forceinline__ void ring_run(const A& a, const B& b, int nk, unsigned char* smem, const RingWave& wv, f32x16 (&acc)[MT][NT]) {
  static_assert(A::SUBS == B::SUBS && A::SUBS % 2 == 0, "stages of both operands hold the same k-steps");
  constexpr int STAGE = ring_stage_bytes<A, B>(), AB = A::PIECES * 1024, S2 = A::SUBS / 2, ROUNDS = A::N + B::N;
  constexpr int LEAST = A::PIECES / RG_WAVES + B::PIECES / RG_WAVES;   // loads of a stage that every wave issues
  constexpr int PRODUCTS = PA + PB - 1, MF = MT * NT * PRODUCTS;       // MFMAs of a k-step
  constexpr int EARLY = ring_early<A, B>(), LATE = ROUNDS - EARLY;
  struct Frags { bf16x8 a[MT][PA], b[NT][PB]; } cur;
  f32x16 small[MT][NT];
  if constexpr (SMALL) ring_zero<MT, NT>(small);
  auto read = [&](Frags& f, const unsigned char* st, int s2) __attribute__((always_inline)) {
    const int sub = 2 * s2 + wv.kg;
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
      for (int p = 0; p < PA; p++) f.a[mt][p] = A::frag(st, sub, wv.wm * MT + mt, p, wv.lane);
#pragma unroll
    for (int nt = 0; nt < NT; nt++)
#pragma unroll
      for (int p = 0; p < PB; p++) f.b[nt][p] = B::frag(st + AB, sub, wv.wn * NT + nt, p, wv.lane);
  };
  // (A with a tail: zeros past the end of k in the last stage)
  auto cut = [&](Frags& f, int kt, int s2) __attribute__((always_inline)) {
    if constexpr (ring_tail<A>(0)) {
      const int left = a.left(kt) - 16 * (2 * s2 + wv.kg) - 4 * (wv.lane >> 5);
      if (a.left(kt) >= 16 * A::SUBS) return;
#pragma unroll
      for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int p = 0; p < PA; p++)
#pragma unroll
          for (int e = 0; e < 8; e++) f.a[mt][p][e] = (e & 3) + 8 * (e >> 2) < left ? f.a[mt][p][e] : (__bf16)0.f;
    }
  };
  const unsigned lds0 = ring_lds(smem);
  int slot = 0;      // of stage kt
  // k-step s2 of stage kt.  STEADY: stage kt + NS exists
  auto step = [&](auto s2_tag, int kt, auto steady_tag) __attribute__((always_inline)) {
    constexpr int s2 = decltype(s2_tag)::value;
    constexpr bool STEADY = decltype(steady_tag)::value, LAST = s2 == S2 - 1;
    const int next = slot + 1 == NS ? 0 : slot + 1, prev = slot == 0 ? NS - 1 : slot - 1;
    Frags nxt = cur;
    if constexpr (LAST) {
      if (STEADY) wait_vmem<(NS - 2) * LEAST>();   // stage kt + 1 has landed: the loads of those behind it may be in flight
      else wait_vmem<0>();
      lds_barrier();
      if (STEADY || kt + 1 < nk) read(nxt, smem + next * STAGE, 0);
      if (!STEADY && kt + 1 == nk - 1) cut(nxt, kt + 1, 0);
    } else {
      read(nxt, smem + slot * STAGE, s2 + 1);
      if (!STEADY && kt == nk - 1) cut(nxt, kt, s2 + 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<MF>([&](auto i_tag) __attribute__((always_inline)) {
      constexpr int i = decltype(i_tag)::value, n = i / (MT * NT), t = PA == 2 && PB == 1 ? n : PRODUCTS - 1 - n, mt = i % (MT * NT) / NT, nt = i % NT;
      constexpr int pa = PA == 2 && PB == 2 ? (t == 1) : PA == 2 ? t : 0, pb = PA == 2 && PB == 2 ? (t == 2) : PB == 2 ? t : 0;
      f32x16& sum = SMALL && t > 0 ? small[mt][nt] : acc[mt][nt];
      sum = mfma32(cur.a[mt][pa], cur.b[nt][pb], sum);
      if constexpr (STEADY) {
        constexpr int N = LAST ? EARLY : s2 == 0 ? LATE : 0;
        static_for<N>([&](auto k_tag) __attribute__((always_inline)) {
          constexpr int k = decltype(k_tag)::value;
          if constexpr ((2 * k + 1) * MF / (2 * N) == i) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (LAST) ring_issue<k>(a, b, kt + NS, lds0 + (unsigned)slot * STAGE, wv);
            else ring_issue<EARLY + k>(a, b, kt - 1 + NS, lds0 + (unsigned)prev * STAGE, wv);
            __builtin_amdgcn_sched_barrier(0);
          }
        });
      }
    });
    cur = nxt;
    if constexpr (LAST) slot = next;
  };
  auto stage = [&](int kt, auto steady) __attribute__((always_inline)) {
    static_for<S2>([&](auto s2) __attribute__((always_inline)) { step(s2, kt, steady); });
  };
  // stage 0 (of the others, at least the loads of NS - 2 are behind it where there are as many)
  if (nk >= NS) wait_vmem<(NS - 2) * LEAST>();
  else wait_vmem<0>();
  lds_barrier();
  read(cur, smem, 0);
  if (nk == 1) cut(cur, 0, 0);
  int kt = 0;
  // (two k-steps a trip at least: the fragments that are read and those in use then change places without copies)
  if constexpr (S2 == 1) {
#pragma unroll 1
    for (; kt + 1 + NS < nk; kt += 2) { stage(kt, std::true_type{}); stage(kt + 1, std::true_type{}); }
  }
#pragma unroll 1
  for (; kt + NS < nk; kt++) stage(kt, std::true_type{});
  if constexpr (LATE > 0) {   // the rounds that a steady step would have issued
    if (nk >= NS) {
      const int prev = slot == 0 ? NS - 1 : slot - 1;
      static_for<LATE>([&](auto k) __attribute__((always_inline)) {
        ring_issue<EARLY + decltype(k)::value>(a, b, nk - 1, lds0 + (unsigned)prev * STAGE, wv);
      });
    }
  }
#pragma unroll 1
  for (; kt < nk; kt++) stage(kt, std::false_type{});
  if constexpr (SMALL) {
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
      for (int nt = 0; nt < NT; nt++) acc[mt][nt] += small[mt][nt];
  }
  __syncthreads();
}

// The two groups' sums: a wave keeps half of its tile, units kg U .. kg U + U - 1 (U = MT NT) of eight registers each, and takes the
// other group's share of them.  Unit u is registers 8 (u % 2) .. of MFMA tile (u / 2 / NT, u / 2 % NT): rows 16 (u % 2) + {0..3, 8..11}
// + 4 h of it.  Begins behind a barrier (ring_run's), ends with one.
template <int MT, int NT>
constexpr int ring_meet_bytes() { return RG_WAVES * MT * NT * 2048; }
// stages that fit: as many as 148 KB hold, at most five
template <class A, class B>
constexpr int ring_stages() {
  constexpr int n = 148 * 1024 / ring_stage_bytes<A, B>();
  return n > 5 ? 5 : n;
}
template <class A, class B>
constexpr int ring_bytes() { return ring_stages<A, B>() * ring_stage_bytes<A, B>(); }
constexpr int ring_max(int a, int b) { return a > b ? a : b; }
template <int MT, int NT>
__device__ __forceinline__ void ring_meet(const f32x16 (&acc)[MT][NT], unsigned char* smem, const RingWave& wv, float (&res)[MT * NT][8]) {
  constexpr int U = MT * NT;
  auto pass = [&](auto kg_tag) __attribute__((always_inline)) {
    constexpr int KG = decltype(kg_tag)::value;
    unsigned char* put = smem + (size_t)(wv.w ^ 4) * U * 2048 + wv.lane * 16;
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int v = (KG ^ 1) * U + u;
#pragma unroll
      for (int q = 0; q < 2; q++) {
        const int r = 8 * (v % 2) + 4 * q;
        const f32x16& t = acc[v / 2 / NT][v / 2 % NT];
        *(f32x4*)(put + (2 * u + q) * 1024) = f32x4{t[r], t[r + 1], t[r + 2], t[r + 3]};
      }
    }
    lds_barrier();
    const unsigned char* get = smem + (size_t)wv.w * U * 2048 + wv.lane * 16;
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int v = KG * U + u;
#pragma unroll
      for (int q = 0; q < 2; q++) {
        const f32x4 o = *(const f32x4*)(get + (2 * u + q) * 1024);
#pragma unroll
        for (int e = 0; e < 4; e++) res[u][4 * q + e] = acc[v / 2 / NT][v / 2 % NT][8 * (v % 2) + 4 * q + e] + o[e];
      }
    }
    lds_barrier();
  };
  if (wv.kg == 0) pass(std::integral_constant<int, 0>{});
  else pass(std::integral_constant<int, 1>{});
}
// MFMA tile and half of the wave's unit u
template <int MT, int NT>
__device__ __forceinline__ void ring_unit(const RingWave& wv, int u, int& mt, int& nt, int& kk) {
  const int v = wv.kg * MT * NT + u;
  mt = v / 2 / NT; nt = v / 2 % NT; kk = v % 2;
}

}  // namespace gc
