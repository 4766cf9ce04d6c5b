// What the bf16 MFMA kernels of the loss path share: operand layouts, direct global->LDS loads, lane exchanges, the
// arguments of the gradient walks.
//
// MFMA operand layouts used throughout (v_mfma_f32_32x32x16_bf16, D = A * B + C, wave of 64):
//   A fragment: lane l holds A[m = l % 32][k = 8 * (l / 32) + 0..7]
//   B fragment: lane l holds B[k = 8 * (l / 32) + 0..7][n = l % 32]
//   C/D:        lane l, register r holds D[m = 8 * (r / 4) + 4 * (l / 32) + r % 4][n = l % 32]
// The reduction over targets is put on the M axis (registers) so that every lane owns one
// anchor column and the softmax statistics need no cross-lane traffic inside a tile.
#pragma once
#include <type_traits>

#include "gc_common.h"
#include "stats_tile.h"

namespace gc {

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// N (1..4) direct global->LDS loads of 16 bytes per lane that share one M0 value.  Load k lands at
// lds_base + 1024 k + lane * 16 and reads gbase + voff[k] + 1024 k: the instruction's immediate
// offset moves both addresses, so callers pass voff[k] with 1024 k already subtracted.  The
// compiler does not see these loads: the reader waits with wait_vmem<N>().
// Every statement below that sets M0 says so in its clobber list.  M0 is a register the backend reserves (it never
// keeps a value of its own there across other code and sets it right before each instruction of its own that needs
// it); the clobber states the write, so that nothing it may ever cache there is assumed to survive.
template <int N>
__device__ __forceinline__ void dma_group(const void* gbase, const unsigned* voff, unsigned lds_base) {
  if constexpr (N == 1) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(voff[0]), "s"(gbase) : "memory", "m0");
  } else if constexpr (N == 2) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024"
                 ::"s"(lds_base), "v"(voff[0]), "v"(voff[1]), "s"(gbase) : "memory", "m0");
  } else if constexpr (N == 3) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4\n\tglobal_load_lds_dwordx4 %2, %4 offset:1024\n\t"
                 "global_load_lds_dwordx4 %3, %4 offset:2048"
                 ::"s"(lds_base), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "s"(gbase) : "memory", "m0");
  } else {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %5\n\tglobal_load_lds_dwordx4 %2, %5 offset:1024\n\t"
                 "global_load_lds_dwordx4 %3, %5 offset:2048\n\tglobal_load_lds_dwordx4 %4, %5 offset:3072"
                 ::"s"(lds_base), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(gbase) : "memory", "m0");
  }
}
// One such load with immediate offset IMM (a multiple of 1024 below 4096): lands at lds_base + IMM +
// lane * 16 and reads gbase + voff + IMM.  No memory clobber: the compiler may move unrelated LDS
// traffic across it; callers order it against the readers of its target with wait_vmem / barriers.
template <int IMM>
__device__ __forceinline__ void dma_piece(const void* gbase, unsigned voff, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"s"(lds_base), "v"(voff), "s"(gbase), "n"(IMM) : "m0");
}
// The same, placed by data dependences instead of fences: the statement claims to rewrite the
// registers pin_a / pin_b (it does not touch them), so it is scheduled after the last reader of
// their old values and before the first reader of the new ones, and nothing else is held up.
// LANES8: only lanes 0-7 load (128 bytes); EXEC is narrowed inside the statement and restored.
template <int IMM, bool LANES8, bool TWO>
__device__ __forceinline__ void dma_piece_pinned(const void* gbase, unsigned voff, unsigned lds_base, u32x4& pin_a, u32x4& pin_b) {
  unsigned pa = pin_a[0], pb = TWO ? pin_b[0] : 0u;
  if constexpr (LANES8) {
    unsigned long long keep;
    if constexpr (TWO)
      asm volatile("s_mov_b64 %2, exec\n\ts_mov_b64 exec, 0xff\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %5 offset:%6\n\ts_mov_b64 exec, %2"
                   : "+v"(pa), "+v"(pb), "=&s"(keep) : "s"(lds_base), "v"(voff), "s"(gbase), "n"(IMM) : "m0");
    else
      asm volatile("s_mov_b64 %1, exec\n\ts_mov_b64 exec, 0xff\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %4 offset:%5\n\ts_mov_b64 exec, %1"
                   : "+v"(pa), "=&s"(keep) : "s"(lds_base), "v"(voff), "s"(gbase), "n"(IMM) : "m0");
  } else {
    if constexpr (TWO)
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %4 offset:%5"
                   : "+v"(pa), "+v"(pb) : "s"(lds_base), "v"(voff), "s"(gbase), "n"(IMM) : "m0");
    else
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3 offset:%4"
                   : "+v"(pa) : "s"(lds_base), "v"(voff), "s"(gbase), "n"(IMM) : "m0");
  }
  pin_a[0] = pa;
  if constexpr (TWO) pin_b[0] = pb;
}
template <int N>
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// __syncthreads() that also waits for this wave's LDS writes by itself.  In loops that write LDS at their end (under a condition)
// and start with a barrier the compiler drops that wait from the barrier: it sees no write pending where the loop is entered.
// A wave behind the barrier has then read a slot before its write, once in some hundred passes over 16384 views.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
}

struct GradArgs {
  const unsigned short* Q;
  const unsigned short* P;
  const int32_t* pos_pad;   // pos_idx copied and padded with -1 to a multiple of 64 rows
  const float* lse2;        // log2-domain log-sum-exp per anchor, padded with +inf
  const float* lse2_t;      // symmetric loss only: the same per target (over the anchors), padded alike
  const float* wexp; const float* wexp_t; const int* wide;   // with it: 2^(-lse2 - 1) of both, and the word that forbids them
  int B, Pn;
  float alpha2, out_scale;
  int mask_self;
  int obQ, nsq, q_stream_len;  // dQ-role workgroups: obQ owner blocks x nsq stream splits
  int obP, nsp, p_stream_len;
  float* dq_out; size_t dq_split_stride;  // split s writes dq_out + s * stride
  float* dp_out; size_t dp_split_stride;
  // online-statistics walk (dQ role, no statistics pass before it): per split and anchor the reference the
  // accumulators are relative to and sum 2^(t - reference); per anchor the positive's logit
  float* on_ref; float* on_l; int* on_idx; float* on_pos;
  float* on_best;  // per split and anchor: the true maximum, written (with on_idx) only when on_argmax is set
  int on_argmax;   // track the true maximum and its first index
  // an anchor per target, as the statistics merge left it, and the word that check_shared_positives raises
  const int32_t* inv; int* shared;
};

// The kernel that sums the partials adds each positive's own term to its dP row through inv[j] (an anchor with
// r_i = j).  That is enough when no two anchors share a target; here every workgroup looks at a slice of the anchors
// and raises *shared when one of them is not the anchor recorded for its target (the sum kernel then scans).
// In three parts, each where the load before it has long arrived: two loads in turn before or behind a kernel's work are 1.5 us.
struct SharedCheck {
  int i, i1, r, seen;
  __device__ __forceinline__ SharedCheck(const GradArgs& ga) : i(0), i1(0), r(-1), seen(0) {
    if (!ga.inv) return;
    const int per = (ga.B + (int)gridDim.x - 1) / (int)gridDim.x;
    i = (int)blockIdx.x * per + (int)threadIdx.x;
    i1 = min(ga.B, ((int)blockIdx.x + 1) * per);
    if (i < i1) r = ga.pos_pad[i];
  }
  __device__ __forceinline__ void look(const GradArgs& ga) {
    seen = i;
    if (r >= 0 && r < ga.Pn) seen = ga.inv[r];
  }
  __device__ __forceinline__ void finish(const GradArgs& ga) {
    if (seen != i) *ga.shared = 1;
    if (i1 - i <= (int)blockDim.x) return;   // (slices longer than the workgroup: the rest of them)
    for (i += (int)blockDim.x; i < i1; i += (int)blockDim.x) {
      r = ga.pos_pad[i];
      if (r >= 0 && r < ga.Pn && ga.inv[r] != i) *ga.shared = 1;
    }
  }
};
__device__ __forceinline__ void check_shared_positives(const GradArgs& ga) {
  SharedCheck c(ga);
  c.look(ga);
  c.finish(ga);
}

// max / sum over the four lanes that share lane % 16 (v_permlane16_swap / v_permlane32_swap give every lane both
// partners' values, so all four lanes end with the same bits)
__device__ __forceinline__ void swap16(unsigned x, unsigned& a, unsigned& b) {
  auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false); a = r[0]; b = r[1];
}
__device__ __forceinline__ void swap32(unsigned x, unsigned& a, unsigned& b) {
  auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false); a = r[0]; b = r[1];
}
__device__ __forceinline__ float max_g16(float x) {
  unsigned a, b;
  swap16(__builtin_bit_cast(unsigned, x), a, b);
  x = fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  swap32(__builtin_bit_cast(unsigned, x), a, b);
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float sum_g16(float x) {
  unsigned a, b;
  swap16(__builtin_bit_cast(unsigned, x), a, b);
  x = __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
  swap32(__builtin_bit_cast(unsigned, x), a, b);
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
// (value, index): larger value wins, ties go to the smaller index
__device__ __forceinline__ void argmax_g16(float& v, int& i) {
  unsigned a, b, ia, ib;
  auto pick = [&]() {
    const float va = __builtin_bit_cast(float, a), vb = __builtin_bit_cast(float, b);
    const bool tb = (vb > va) || (vb == va && (int)ib < (int)ia);
    v = tb ? vb : va; i = tb ? (int)ib : (int)ia;
  };
  swap16(__builtin_bit_cast(unsigned, v), a, b); swap16((unsigned)i, ia, ib); pick();
  swap32(__builtin_bit_cast(unsigned, v), a, b); swap32((unsigned)i, ia, ib); pick();
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {  // f(integral_constant<int, I>) for I = 0 .. N-1
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Sum (or maximum) of 16 registers, each over the 32 lanes of its half-wave, by halving: every exchange combines two
// registers into one, so they cost about 40 operations, not 160.  The result of register r is in the lanes whose
// bits 4, 3, 2, 1 spell bits 0, 1, 2, 3 of r (bit 0 of the lane: a copy).
template <bool MAX>
__device__ __forceinline__ float lane_op(float a, float b) { return MAX ? fmaxf(a, b) : a + b; }
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
constexpr int kRor8 = 0x128, kHalfMirror = 0x141, kXor2 = 0x4e, kXor1 = 0xb1;   // row_ror:8, row_half_mirror, quad_perm
template <bool MAX>
__device__ __forceinline__ float reduce16_lanes32(const float (&v)[16], int lane) {
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
  float u[8], w[4], x[2];
#pragma unroll
  for (int k = 0; k < 8; k++) {
    auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v[2 * k]), __builtin_bit_cast(unsigned, v[2 * k + 1]), false, false);
    u[k] = lane_op<MAX>(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
  }
#pragma unroll
  for (int k = 0; k < 4; k++) w[k] = lane_op<MAX>(b3 ? u[2 * k + 1] : u[2 * k], dpp<kRor8>(b3 ? u[2 * k] : u[2 * k + 1]));
#pragma unroll
  for (int k = 0; k < 2; k++) x[k] = lane_op<MAX>(b2 ? w[2 * k + 1] : w[2 * k], dpp<kHalfMirror>(b2 ? w[2 * k] : w[2 * k + 1]));
  const float y = lane_op<MAX>(b1 ? x[1] : x[0], dpp<kXor2>(b1 ? x[0] : x[1]));
  return lane_op<MAX>(y, dpp<kXor1>(y));
}
__device__ __forceinline__ int reduce16_reg_of(int lane) { return ((lane >> 4) & 1) | ((lane >> 2) & 2) | (lane & 4) | ((lane << 2) & 8); }
// ... and back: what reduce16_lanes32 left for register R, in every lane of the half-wave (ds_swizzle: all from one lane)
template <int R>
__device__ __forceinline__ float reduce16_spread(float x) {
  constexpr int from = ((R & 1) << 4) | ((R & 2) << 2) | (R & 4) | ((R & 8) >> 2);
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x), from << 5));
}
// maximum over the 32 lanes of the half-wave, in every lane
__device__ __forceinline__ float max_lanes32(float x) {
  unsigned a, b;
  swap16(__builtin_bit_cast(unsigned, x), a, b);
  x = fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  x = fmaxf(x, dpp<kRor8>(x));
  x = fmaxf(x, dpp<kHalfMirror>(x));
  x = fmaxf(x, dpp<kXor2>(x));
  return fmaxf(x, dpp<kXor1>(x));
}

// Statistics of both sides of a score matrix from one pass over its scores (the symmetric forms): sums of 2^t per row (lanes)
// and per column of a tile with the reference 0.  A tile whose sums all lie in these bounds has lost nothing: what 2^t flushes
// is below 2^-126.  Any other tile (and one with masked scores) takes the maxima of its rows and columns as references.
// (stats_mfma_kernel: a column's maximum goes back to its lanes by ds_swizzle, and a wave tries the reference 0 again once the
// references of a tile allow it.  4096 views of 256, logits far beyond: about 30 us before that, 20.5 so, 16.5 with the reference 0.)
constexpr float kBothMin = 0x1p-60f, kBothMax = 0x1p100f, kBothMinLog2 = -60.f, kBothMaxLog2 = 100.f;
struct StatsArgs {
  const unsigned short* Q; const unsigned short* P; const int32_t* pos_idx;
  int B, Pn, d;              // owners (lanes), streamed rows
  int n_ablk, cols_per_split, mask_self;
  float alpha2;
  // partials (maximum, sum relative to it): [slot][row].  Rows: slot = range of the streamed rows; columns: slot = owner block
  float* row_m; float* row_l; int* row_idx; float* col_m; float* col_l;
  float* pos_t;
  // statistics of both sides: word that the merge may raise; symmetric loss: inv[r_i] = i for every valid r_i (whatever the
  // workspace held stays elsewhere: whoever reads an entry checks it)
  int* zero; int32_t* inv;
};
__device__ __forceinline__ void both_begin(const StatsArgs& g) {
  const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (t == 0) *g.zero = 0;
  if (!g.inv) return;
  for (int i = t; i < g.B; i += (int)(gridDim.x * blockDim.x)) {
    const int r = g.pos_idx[i];
    if (r >= 0 && r < g.Pn) g.inv[r] = i;
  }
}
// TRI: tasks are block 0's ranges of the rows from the block's first one on, then block 1's, ...
__device__ __forceinline__ int tri_task(int task, int n, int block, int len, int& ablk) {
  for (ablk = 0;; ablk++) {
    const int c = (n - ablk * block + len - 1) / len;
    if (task < c) return task;
    task -= c;
  }
}
hipError_t launch_stats128_both(const StatsArgs& g, bool triangle, int nwg, hipStream_t stream);

// d = 128 (loss_mfma128.hip)
constexpr int G1_OWN = 128;   // owner rows per workgroup of the gradient pass
hipError_t launch_stats128(const LossArgs& a, const LossPlan& pl);
hipError_t grad128_launch(const GradArgs& ga, int nwg, hipStream_t stream);

// symmetric forms, d >= 256 (loss_mfma_sym.hip)
hipError_t grad_sym_launch(const GradArgs& ga, int d, int nwg, hipStream_t stream);

// few scores (loss_few.hip)
hipError_t grad_few_launch(const GradArgs& ga, const FewMerge& fm, int d, int nwg, hipStream_t stream);

}  // namespace gc
