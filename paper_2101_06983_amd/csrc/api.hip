// C ABI of the library: argument checks, workspace planning and kernel sequencing.
// Every check happens before the first HIP call of an entry point.
#include <cmath>
#include <cstring>
#include <mutex>

#include "gc_common.h"

// The workspace of gc_loss_and_rep_grad_bf16_static (see static_scratch below): a fixed array in the device image.
static __device__ __align__(256) unsigned char scratch[GC_STATIC_SCRATCH_BYTES];

namespace gc {

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Compute units of the current device (sizes grids and the stream splits of the workspace plan), asked once per
// process; without a device (the host-only checks of the test-suite) the MI355X count.
int num_cu() {
  static int cached = 0;
  if (cached > 0) return cached;
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
    cached = n;
  else
    cached = kNumCUDefault;
  (void)hipGetLastError();
  return cached;
}

// rows per workgroup of the gradient pass when every compute unit gets one and all get an equal share, at least 256
static long long equal_share(long long rows) {
  const long long L = (rows + num_cu() - 1) / num_cu();
  return L < 256 ? 256 : (L + 31) / 32 * 32;
}
// few, parts_limit, equal: ROUTE_MFMA.  few: small statistics tiles where the scores are few.  Splits: the fastest whose
// partials stay below parts_limit bytes, or (equal) the fewest that give every compute unit an equal share of the rows.
// lean: 1: as many splits of the statistics as with blocks of 256, two of which share no compute unit; 2: and a second round of
// workgroups priced as a whole one, which takes fewer splits.
// now: the gradient kernels as they are.  Without it, as in the plans for a limited workspace, the blocks and costs that decide
// the splits are those of the walks with 64 rows (d = 128: 256 rows), so that the sizes taken do not change with the kernels.
static LossPlan make_loss_plan_for(int B, int P, int d, gc_dtype dt, bool ntxent, int route, int max_splits, bool few, double parts_limit,
                                   bool equal = false, bool now = false, int lean = 0) {
  LossPlan pl{};
  const int kNumCU = num_cu();
  pl.route = route;
  pl.use_mfma = route == ROUTE_MFMA ? 1 : 0;
  if (route == ROUTE_PLANES) {
    plan_planes(pl, B, P, d, dt, max_splits);
  } else if (pl.use_mfma) {
    if (few && (long long)B * P <= (1ll << 20)) {   // where the line lies: see stats_small_kernel
      pl.stat_tile = kStatTile;
      const int tiles = ceil_div(P, kStatTile), per = ceil_div(tiles, 64);   // the merge kernel combines at most 64 splits
      pl.stat_cols_per_split = per * kStatTile;
      pl.stat_splits = ceil_div(tiles, per);
    } else {
      // two workgroups to a CU, blocks of 256 anchors at d = 128; without `few`: one of 256 x 256 scores, for fewer partials
      const bool mid = few && !lean && d > 128 && stats_block(B, P, d) == kStatBlock;
      const int T = mid ? kStatBlock : 256, n_ablk = ceil_div(B, T), tiles = ceil_div(P, T);
      int splits = ceil_div(mid || d == 128 ? 2 * kNumCU : kNumCU, n_ablk);
      if (splits > 64) splits = 64;
      if (splits > tiles) splits = tiles;
      if (splits < 1) splits = 1;
      if (mid && n_ablk * ceil_div(tiles, ceil_div(tiles, splits)) > 2 * kNumCU) {
        // A few workgroups more than run at once can be a second round (544 at 8642 x 7000 x 512: 115 us for the loss alone; 7 splits,
        // 476 workgroups: 79).  The splits with the least time, in tiles and half a one for a workgroup's start: whole rounds, then
        // the last split's workgroups, which have `rest` tiles, on the places that are left and, those beyond, behind one another.
        // (A multiple of 8 workgroups is dealt to the XCDs in contiguous ranges: most of them then have no short ones, and one more
        // than they have places for is a round, 0.65 of one where the places are half empty.)
        double best = 0;
        for (int s = 1; s <= 64 && s <= tiles; s++) {
          const int cap = 2 * kNumCU, per = ceil_div(tiles, s), full = ceil_div(tiles, per) - 1, rest = tiles - full * per;
          const int in = n_ablk * full % cap, left = in + n_ablk - cap;
          const double first = in ? per + 0.5 : rest + 0.5, behind = left > 0 ? (rest + 0.5) * (1 + 0.9 * ceil_div(left, cap)) : 0;
          double t = (per + 0.5) * (n_ablk * full / cap) + (first > behind ? first : behind);
          const int wgs = n_ablk * (full + 1), last = wgs % cap;
          if (wgs % 8 == 0) t = (per + 0.5) * (wgs / cap + (last == 0 ? 0. : last <= cap / 2 ? 0.65 : 1.));
          if (best == 0 || t < best) { best = t; splits = s; }
        }
      }
      pl.stat_cols_per_split = ceil_div(tiles, splits) * T;
      pl.stat_splits = ceil_div(P, pl.stat_cols_per_split);
    }
    // owner rows per workgroup of the gradient kernel for this width
    const bool wide128 = d == 128 && !now;
    // calls with few scores have a gradient kernel of their own (see loss_few.hip); limited workspaces do not
    pl.few_grad = pl.stat_tile && now;
    const int own = pl.few_grad ? kFewOwn : d > 128 ? 64 : wide128 ? 256 : 128;
    const long long obQ = ceil_div(B, own), obP = ceil_div(P, own);
    // NT-Xent on these kernels is one walk (the score matrix is symmetric: see launch_grad_mfma)
    pl.one_walk = ntxent ? 1 : 0;
    // Gradient pass: every workgroup streams about the same number of rows, L.  Its time is ceil(workgroups / CUs) rounds (a
    // compute unit holds one, of the d = 256 kernel two) of a fixed part and a part per streamed row, and every split of an output is a partial that is
    // written and read again.  The splits that make L and the rounds come out even are tried: an equal share of the rows
    // per compute unit can give a few workgroups more than there are CUs, and with them a second round (258 workgroups
    // at 1021 x 4099 x 384: 46 us, 29 with 242), and few scores leave the CUs idle (6 workgroups at 128 x 256 x 768: 21 us,
    // 15.6 with 32).
    // Measured: 14 us and 0.03 to 0.05 us per row at d = 768; 8 and 0.022 at d = 128; the kernel for few scores 7 and 0.02 to
    // 0.047; partials about 4 TB/s.
    // (Two workgroups of the d = 128 and d = 256 kernels share a compute unit, each at some 70 % of its speed.)
    const bool two128 = d == 128 && !wide128;
    const double row_us = pl.few_grad ? 0.02 + 0.027 * d / 768.0 : wide128 ? 0.031 : two128 ? 0.022 : 0.015 + 0.035 * d / 768.0, fixed_us = pl.few_grad ? 7.0 : two128 ? 8.0 : 14.0;
    const int per_cu = d <= 256 && !wide128 ? 2 : 1;
    auto len_of = [](int n, int ns) { return (ceil_div(n, ns) + 31) / 32 * 32; };
    auto parts_bytes = [&](int nsq, int nsp) { return ((double)nsq * B + (double)nsp * P) * d * 4; };
    double best_us = 0;
    auto consider = [&](int L, bool walk_q, bool walk_p, int& bq, int& lq, int& bp, int& lp) {
      const int nsq = walk_q ? (ceil_div(P, L) > 16 ? 16 : ceil_div(P, L)) : 0, nsp = walk_p ? (ceil_div(B, L) > 16 ? 16 : ceil_div(B, L)) : 0;
      const int q = walk_q ? len_of(P, nsq) : 0, p = walk_p ? len_of(B, nsp) : 0;
      const long long n = (walk_q ? obQ * ceil_div(P, q) : 0) + (walk_p ? obP * ceil_div(B, p) : 0);
      const double parts = parts_bytes(walk_q ? ceil_div(P, q) : 0, walk_p ? ceil_div(B, p) : 0);
      const double both = n > kNumCU && per_cu == 2 ? 1.4 : 1.0;
      const long long slots = (long long)per_cu * kNumCU;
      double walk_us = (double)((n + slots - 1) / slots) * (fixed_us + row_us * both * (q > p ? q : p));
      if (pl.few_grad && n > slots && lean < 2) {
        // The kernel for few scores starts the longer walks first: the longer of one of them, in as many rounds as they take, and an
        // equal share of all the work with one of the shorter walks behind it.  (A whole round of the longest for the last few short
        // walks sent 46 x 7607 x 768, 16 walks of 480 rows and 238 of 46, to 8 of 960: 71.4 us a call, 56.7 so, 64.0 with the long walks.)
        const double uq = walk_q ? fixed_us + row_us * both * q : 0, up = walk_p ? fixed_us + row_us * both * p : 0;
        const long long wq = walk_q ? obQ * ceil_div(P, q) : 0, wp = n - wq, wl = uq > up ? wq : wp;
        const double longest = uq > up ? uq : up, alone = longest * (double)((wl + slots - 1) / slots);
        const double share = (wq * uq + wp * up) / (double)slots + (wq == 0 || wp == 0 ? 0 : uq < up ? uq : up);
        walk_us = alone > share ? alone : share;
      }
      const double us = walk_us + 2.0 * parts / 4e6;
      if (parts <= parts_limit && (best_us == 0 || us < best_us)) {
        best_us = us;
        if (walk_q) { bq = ceil_div(P, q); lq = q; }
        if (walk_p) { bp = ceil_div(B, p); lp = p; }
      }
    };
    auto search = [&](bool walk_q, bool walk_p, int& bq, int& lq, int& bp, int& lp) {
      best_us = 0;
      for (int ns = 1; ns <= 16; ns++) {
        if (walk_q) consider(len_of(P, ns), walk_q, walk_p, bq, lq, bp, lp);
        if (walk_p) consider(len_of(B, ns), walk_q, walk_p, bq, lq, bp, lp);
      }
      if (best_us == 0) consider(B > P ? len_of(B, 1) : len_of(P, 1), walk_q, walk_p, bq, lq, bp, lp);
    };
    auto share = [&](long long rows, int n, int& ns, int& len) {   // rows: those that all workgroups stream together
      const long long L = equal_share(rows);
      ns = (int)((n + L - 1) / L > 16 ? 16 : (n + L - 1) / L);
      len = len_of(n, ns);
      ns = ceil_div(n, len);
    };
    pl.nsq = pl.nsp = 1; pl.q_stream_len = len_of(P, 1); pl.p_stream_len = len_of(B, 1);
    const long long rows_q = obQ * P, rows_p = obP * B, rows_all = pl.one_walk ? rows_q : rows_q + rows_p;
    if (equal) {
      share(rows_all, P, pl.nsq, pl.q_stream_len);
      share(rows_all, B, pl.nsp, pl.p_stream_len);
    } else {
      search(true, !pl.one_walk, pl.nsq, pl.q_stream_len, pl.nsp, pl.p_stream_len);
    }
    if (pl.one_walk) { pl.nsp = 1; pl.p_stream_len = B; }
    if (pl.few_grad && d > 128) {
      auto rounds = [&](int n, int own_rows, int splits) { return ceil_div(ceil_div(n, own_rows) * splits, per_cu * kNumCU); };
      pl.few_not_q = rounds(B, kFewOwn, pl.nsq) > 1 && rounds(B, 64, pl.nsq) == 1;
      pl.few_not_p = rounds(P, kFewOwn, pl.nsp) > 1 && rounds(P, 64, pl.nsp) == 1;
    }
    pl.few_merge = pl.few_grad && !ntxent && pl.p_stream_len <= kFewMergeRows && pl.p_stream_len * pl.stat_splits <= kFewMergeEntries;
    // fused mode (workspace is planned for it wherever it can run; fused_auto says where it is also the faster one):
    // each walk is a launch of its own and has to fill the GPU alone
    // (it pays where the statistics pass it replaces is expensive against the extra partial sums.  A call with it / with
    // the statistics pass, us:    4096 x 4096   1024 x 16384   4096 x 6000   4096 x 8192   2048 x 16384
    //   d = 256                   101 / 83      101 / 82       240 / 151     165 / 135     166 / 136
    //   d = 384                   112 / 108     118 / 117      160 / 176     183 / 187     187 / 197
    //   d = 512                   131 / 130     141 / 145      188 / 206     212 / 221     220 / 243
    //   d = 768                   165 / 158     178 / 184      224 / 248     259 / 273     263 / 295
    // and far slower below 2^24 scores, where launches and partials dominate)
    pl.fused = (d >= 256 && !ntxent) ? 1 : 0;
    pl.fused_auto = (pl.fused && d >= 384 && (long long)B * P >= (1ll << 24)) ? 1 : 0;
    if (pl.fused) {
      // (where only a flag asks for it, the splits, and so the workspace, of the other sequence)
      pl.fz_nsq = pl.nsq; pl.fz_q_stream_len = pl.q_stream_len;
      pl.fz_nsp = pl.nsp; pl.fz_p_stream_len = pl.p_stream_len;
      int unused = 0;
      if (pl.fused_auto && equal) {
        share(rows_q, P, pl.fz_nsq, pl.fz_q_stream_len);
        share(rows_p, B, pl.fz_nsp, pl.fz_p_stream_len);
      } else if (pl.fused_auto) {
        search(true, false, pl.fz_nsq, pl.fz_q_stream_len, unused, unused);
        search(false, true, unused, unused, pl.fz_nsp, pl.fz_p_stream_len);
      }
    }
  } else {
    const int blocks = ceil_div(B, 16), tiles = ceil_div(P, 16);
    int splits = ceil_div(4 * kNumCU, blocks);
    if (splits > 64) splits = 64;
    if (splits > tiles) splits = tiles;
    if (splits < 1) splits = 1;
    pl.stat_cols_per_split = ceil_div(tiles, splits) * 16;
    pl.stat_splits = ceil_div(P, pl.stat_cols_per_split);
    pl.nsq = pl.nsp = 1;
    pl.q_stream_len = P;
    pl.p_stream_len = B;
  }
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
  pl.off_err = take(256);
  const int stat_parts = pl.stat_splits > pl.fz_nsq ? pl.stat_splits : pl.fz_nsq;   // fz_* are 0 outside fused mode
  pl.off_part_m = take((size_t)stat_parts * B * 4);
  pl.off_part_l = take((size_t)stat_parts * B * 4);
  pl.off_part_idx = take((size_t)stat_parts * B * 4);
  pl.b_pad = route == ROUTE_PLANES ? (B + 127) / 128 * 128 : (B + 63) / 64 * 64;
  pl.off_pos = take((size_t)(route == ROUTE_PLANES ? pl.b_pad : B) * 4);
  pl.off_lse2 = take((size_t)pl.b_pad * 4);
  pl.off_pos_pad = take((size_t)pl.b_pad * 4);
  pl.off_rowloss = take((size_t)B * 4);
  // an anchor per target (see PosFix); among the statistics: everything below off_dq_part is what a call that only
  // forms statistics touches (the symmetric loss sizes its second workspace by that)
  pl.off_inv = take(pl.use_mfma ? (size_t)P * 4 : 0);
  int dq_parts = (pl.nsq > 1 || ntxent) ? pl.nsq : 0, dp_parts = ((pl.nsp > 1 || ntxent) && !pl.one_walk) ? pl.nsp : 0;
  if (pl.use_mfma && !ntxent) {  // the MFMA walks always write partials: the kernel that sums them adds the
    if (dq_parts < 1) dq_parts = 1;  // positive's term in fp32 (PosFix) and rounds a bf16 cache
    if (dp_parts < 1) dp_parts = 1;
  }
  if (pl.fused) {
    if (pl.fz_nsq > dq_parts) dq_parts = pl.fz_nsq;            // the online walk always writes partials
    if (pl.fz_nsp > 1 && pl.fz_nsp > dp_parts) dp_parts = pl.fz_nsp;
  }
  pl.px_stride_q = align_up((size_t)B * d, 4);
  pl.px_stride_p = align_up((size_t)P * d, 4);
  pl.off_dq_part = take((size_t)dq_parts * (route == ROUTE_PLANES ? pl.px_stride_q : (size_t)B * d) * 4);
  pl.off_dp_part = take((size_t)dp_parts * (route == ROUTE_PLANES ? pl.px_stride_p : (size_t)P * d) * 4);
  if (route == ROUTE_PLANES) {
    const size_t per_row = (size_t)pl.px_KS * 16 * 2 * pl.np;
    pl.off_qk = take(pl.px_rows_q * per_row);
    pl.off_qt = take(pl.px_rows_q * per_row);
    pl.off_pk = take(pl.px_rows_p * per_row);
    pl.off_pt = take(pl.px_rows_p * per_row);
  }
  pl.off_on_ref = take((size_t)pl.fz_nsq * B * 4);
  pl.off_pos_idx = take(ntxent ? (size_t)B * 4 : 0);
  pl.total = off;
  return pl;
}
// what the packed inputs and partials may take without being asked about (the rest of a 288 GB card is the caller's)
constexpr size_t kPlanesMaxBytes = (size_t)32 << 30;
static double parts_bytes_of(const LossPlan& pl, int B, int P, int d) { return ((double)pl.nsq * B + (double)pl.nsp * P) * d * 4; }
// partials of an equal share of the rows per compute unit
static double equal_parts(int B, int P, int d, bool ntxent) {
  const int own = (d == 128) ? 256 : 64;
  const long long obQ = ceil_div(B, own), obP = ceil_div(P, own), L = equal_share(obQ * P + (ntxent ? 0 : obP * B));
  return ((double)((P + L - 1) / L) * B + (double)((B + L - 1) / L) * P) * d * 4;
}
// Which bf16 shapes of the MFMA route the entry point with the fixed array takes is decided by the plans without `now`, so that
// it does not change with the kernels.  (Two searches over the splits, some 4 us of host time each:
// the other entry points do not ask, unless a plan of theirs has to be made to fit.)
static bool static_takes(int B, int P, int d) {
  auto total = [&](bool few, double limit) { return make_loss_plan_for(B, P, d, GC_BF16, false, ROUTE_MFMA, 16, few, limit, false).total; };
  const size_t fixed = (size_t)GC_STATIC_SCRATCH_BYTES;
  return total(true, 1e300) <= fixed || total(false, equal_parts(B, P, d, false)) <= fixed;
}
// The plan with the first in order of speed whose workspace `fits` takes; if it takes none, the last.
template <class Fits>
static LossPlan choose_plan(int B, int P, int d, gc_dtype dt, bool ntxent, Fits fits) {
  if (dt == GC_BF16 && d % 128 == 0 && d >= 128 && d <= 768) {
    const double parts = equal_parts(B, P, d, ntxent);
    auto plan = [&](bool few, double parts_limit, bool equal, bool now = false, int lean = 0) {
      return make_loss_plan_for(B, P, d, dt, ntxent, ROUTE_MFMA, 16, few, parts_limit, equal, now, lean);
    };
    const size_t fixed = (size_t)GC_STATIC_SCRATCH_BYTES;
    auto first = [&](int lean) {
      LossPlan pl = plan(true, 1e300, false, true, lean);
      if (pl.total > fixed && pl.few_grad && static_takes(B, P, d)) {   // fewer splits of the same kernel, if they fit it
        const double now_parts = parts_bytes_of(pl, B, P, d), room = (double)fixed - ((double)pl.total - now_parts);
        const LossPlan less = plan(true, room, false, true, lean);
        if (less.total <= fixed) pl = less;
      }
      if (pl.total > fixed) {
        // the shapes that the entry point with the fixed array takes do not depend on the splits: those that fit with an
        // equal share of the rows per compute unit, at least 256 of them, get splits that fit
        const LossPlan share = plan(false, parts, false);
        if (share.total <= fixed) {
          const LossPlan both = plan(true, parts, false);
          pl = both.total <= fixed ? both : share;
        }
      }
      return pl;
    };
    LossPlan pl = first(0);
    if (fits(pl)) return pl;
    // What a call needs at least does not change with the kernels: one of these has to fit.
    const LossPlan least[] = {first(2), plan(true, parts, false), plan(false, parts, false), plan(false, parts, true)};
    const LossPlan* fit = nullptr;
    for (const LossPlan& l : least)
      if (!fit && fits(l)) fit = &l;
    if (!fit) return least[3];
    // Then the first plan again with fewer splits.  (A workspace that an earlier version named is often just short of the present one:
    // with the plans above 5750 x 10557 x 384 took 388 us a call in it and 1621 x 13677 x 256, dq alone, 114; 330 and 74 so.)
    const double now_bytes = (double)(pl.off_on_ref - pl.off_dq_part);
    for (const double part : {1., 0.95, 0.85, 0.7, 0.55, 0.4, 0.3, 0.2, 0.1}) {
      pl = plan(true, part * now_bytes, false, true, 1);
      if (pl.total < fit->total) pl.total = fit->total;   // (asked again with this plan's size as the limit: the same plan)
      if (fits(pl)) return pl;
    }
    return *fit;
  }
  if (tiny_fits(B, P, d)) return make_loss_plan_for(B, P, d, dt, ntxent, ROUTE_TINY, 1, false, 0.);
  for (int splits = 16; splits >= 1; splits /= 2) {
    const LossPlan pl = make_loss_plan_for(B, P, d, dt, ntxent, ROUTE_PLANES, splits, false, 0.);
    if (pl.total <= kPlanesMaxBytes && fits(pl)) return pl;
  }
  return make_loss_plan_for(B, P, d, dt, ntxent, ROUTE_GENERAL, 1, false, 0.);
}

// A plan depends on nothing but these arguments (and num_cu(), one number per process); the last ones of a thread, without a limit and with one, are kept (the
// search over the splits is some microseconds of host time, and a program asks for the same plan call after call).
LossPlan make_loss_plan(int B, int P, int d, gc_dtype dt, bool ntxent, size_t limit) {
  struct Kept {
    int B = 0, P, d; gc_dtype dt; bool ntxent; size_t limit; LossPlan pl;
    const LossPlan& get(int B_, int P_, int d_, gc_dtype dt_, bool ntxent_, size_t limit_) {
      if (B != B_ || P != P_ || d != d_ || dt != dt_ || ntxent != ntxent_ || limit != limit_) {
        pl = choose_plan(B_, P_, d_, dt_, ntxent_, [limit_](const LossPlan& p) { return p.total <= limit_; });
        B = B_; P = P_; d = d_; dt = dt_; ntxent = ntxent_; limit = limit_;
      }
      return pl;
    }
  };
  static thread_local Kept whole, limited;
  const LossPlan& pl = whole.get(B, P, d, dt, ntxent, (size_t)-1);
  return pl.total <= limit ? pl : limited.get(B, P, d, dt, ntxent, limit);
}

static bool shape_ok(int B, int P, int d) {
  if (B < 1 || P < 1 || d < 1) return false;
  if ((long long)B * d > (1ll << 40) || (long long)P * d > (1ll << 40)) return false;
  return true;
}

// per-device buffer behind the entry points that take no workspace
static std::mutex g_ws_mutex;
static void* g_ws_ptr[64];
static size_t g_ws_bytes[64];
// A buffer that a captured call has used belongs to the recorded graph as well: growing leaves it allocated (until the
// process ends: nothing says when the last graph is gone)
static bool g_ws_recorded[64];
constexpr int kMaxKept = 32;   // (more are kept all the same, but gc_check_async_error does not read them)
static void* g_ws_kept[64][kMaxKept];
static int g_ws_nkept[64];

// GC_OK with the buffer in *out; else what there is in *out and *have, and GC_ERR_UNSUPPORTED where a capture forbids
// growing it, GC_ERR_HIP where the device has no room for `need`.
static int own_workspace(size_t need, hipStream_t stream, void** out, size_t* have) {
  int dev = 0;
  *out = nullptr;
  *have = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return GC_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_ws_mutex);
  int rc = GC_OK;
  if (g_ws_bytes[dev] < need) {
    // growing allocates, and frees the old buffer (which waits for the device): neither is legal while the
    // caller's stream is being captured into a graph
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) { (void)hipGetLastError(); cap = hipStreamCaptureStatusNone; }
    size_t room = need, total = 0;
    if (cap != hipStreamCaptureStatusNone) rc = GC_ERR_UNSUPPORTED;
    else if (hipMemGetInfo(&room, &total) != hipSuccess) { (void)hipGetLastError(); room = need; }
    // room that there cannot be is not asked for: the old buffer then stays in use, call after call
    if (rc == GC_OK && room + (g_ws_recorded[dev] ? 0 : g_ws_bytes[dev]) < need) rc = GC_ERR_HIP;
    if (rc == GC_OK) {
      if (g_ws_ptr[dev] && g_ws_recorded[dev]) {
        if (g_ws_nkept[dev] < kMaxKept) g_ws_kept[dev][g_ws_nkept[dev]++] = g_ws_ptr[dev];
      } else if (g_ws_ptr[dev]) {
        (void)hipFree(g_ws_ptr[dev]);  // waits for work that still uses it
      }
      g_ws_ptr[dev] = nullptr;
      g_ws_bytes[dev] = 0;
      g_ws_recorded[dev] = false;
      for (const size_t sz : {align_up(need + need / 4, 1 << 20), align_up(need, 4096)}) {
        if (hipMalloc(&g_ws_ptr[dev], sz) == hipSuccess) { g_ws_bytes[dev] = sz; break; }
        (void)hipGetLastError();   // a refused allocation is no error of the launches that follow
        g_ws_ptr[dev] = nullptr;
      }
      if (!g_ws_ptr[dev]) rc = GC_ERR_HIP;
    }
  }
  *out = g_ws_ptr[dev];
  *have = g_ws_bytes[dev];
  return rc;
}

// Calls that share the library's buffer from different streams are put in order: each call leaves an event behind
// its last kernel, and a call on another stream waits for it first.  (Not while a stream is being captured: an
// event of ordinary work cannot be waited for inside a capture; a captured call must not overlap with other calls
// on the buffer.)
static hipEvent_t g_ws_done[64];
static hipStream_t g_ws_last[64];
static bool g_ws_used[64];
static bool is_capturing(hipStream_t stream) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess) { (void)hipGetLastError(); return false; }
  return cap != hipStreamCaptureStatusNone;
}
// (The device and the state of the stream are asked for once a call: of the 9 us of host time that a call with a handful of scores
// spends in here, each question is 0.2 to 0.4.)
struct OwnCall { int dev; bool capturing; };
static int own_workspace_enter(hipStream_t stream, OwnCall& c) {
  c.dev = 0;
  if (hipGetDevice(&c.dev) != hipSuccess || c.dev < 0 || c.dev >= 64) return GC_ERR_HIP;
  c.capturing = is_capturing(stream);
  std::lock_guard<std::mutex> lock(g_ws_mutex);
  if (c.capturing) { g_ws_recorded[c.dev] = true; return GC_OK; }
  if (g_ws_used[c.dev] && g_ws_last[c.dev] != stream && hipStreamWaitEvent(stream, g_ws_done[c.dev], 0) != hipSuccess) return GC_ERR_HIP;
  return GC_OK;
}
static int own_workspace_leave(hipStream_t stream, const OwnCall& c) {
  if (c.capturing) return GC_OK;
  std::lock_guard<std::mutex> lock(g_ws_mutex);
  if (!g_ws_done[c.dev] && hipEventCreateWithFlags(&g_ws_done[c.dev], hipEventDisableTiming) != hipSuccess) return GC_ERR_HIP;
  if (hipEventRecord(g_ws_done[c.dev], stream) != hipSuccess) return GC_ERR_HIP;
  g_ws_last[c.dev] = stream;
  g_ws_used[c.dev] = true;
  return GC_OK;
}

// ---- the workspace of the entry point that allocates nothing: a fixed array in the device image ---------------
// One copy per GPU, at an address of its own.  Host code never uses the array's name as an address (on the host
// it is only a handle for the lookup): the address is asked for once per device, with that device current, and
// kept; kernels get it as an ordinary pointer argument, exactly as they get a caller's workspace.
static void* g_scratch_ptr[64];   // per device: what hipGetSymbolAddress answered (under g_ws_mutex)

static int static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return GC_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_ws_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return GC_ERR_HIP; }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return GC_OK;
}

// ---- measurement aid: HIP events around the phases of the loss path ------------------------------
struct Profile {
  bool on = false;
  int max_calls = 0, calls = 0;
  hipEvent_t* ev = nullptr;  // [max_calls][kMarks]
};
constexpr int kMarks = 5;  // start | after stats | after merge | after gradient kernel | after partial sums
static Profile g_prof;

static void prof_mark(int call, int mark, hipStream_t s) {
  if (g_prof.on && call < g_prof.max_calls) (void)hipEventRecord(g_prof.ev[call * kMarks + mark], s);
}
void prof_mark_grad_kernel_done(hipStream_t s) { prof_mark(g_prof.calls, 3, s); }
bool prof_active() { return g_prof.on; }

static int run_loss(const LossArgs& a_in, const LossPlan& pl) {
  LossArgs a = a_in;
  if (!a.ws2) a.ws2 = a.ws;
  // does the gradient pass of this call end in a sum of split partials that takes the row losses along?
  a.loss_with_partials = pl.route != ROUTE_GENERAL && (a.sym[0] || (!a.lse2_t && !a.defer_loss_sum)) && (a.dz || a.dq || a.dp);
  const int call = g_prof.calls;
  prof_mark(call, 0, a.stream);
  hipError_t e;
  if (pl.route == ROUTE_TINY) {   // everything is the first phase
    if (launch_loss_tiny(a, pl) != hipSuccess) return GC_ERR_HIP;
    for (int mark = 1; mark < kMarks; mark++) prof_mark(call, mark, a.stream);
    if (g_prof.on) g_prof.calls++;
    return GC_OK;
  }
  const bool want_online = (a.flags & GC_PATH_ONLINE) || (pl.fused_auto && !(a.flags & GC_PATH_STATS_PASS));
  if (pl.fused && want_online && a.dq && !a.dz && !a.lse2_t) {
    // fused mode: online-statistics dQ walk | merge of its splits (lse2, row losses, dQ) | dP walk | partial sums
    e = launch_grad_online(a, pl);
    if (e != hipSuccess) return GC_ERR_HIP;
    prof_mark(call, 1, a.stream);
    e = launch_online_finish(a, pl);
    if (e != hipSuccess) return GC_ERR_HIP;
    prof_mark(call, 2, a.stream);
    bool loss_done = false;
    if (a.dp) {
      LossArgs b = a;
      LossPlan pb = pl;
      b.dq = nullptr;
      pb.nsp = pl.fz_nsp; pb.p_stream_len = pl.fz_p_stream_len;
      b.loss_with_partials = true;   // the dP walk always ends in the sum of its partials
      loss_done = true;
      e = launch_grad_mfma(b, pb);   // records mark 3 after the walk
      if (e != hipSuccess) return GC_ERR_HIP;
    } else {
      prof_mark(call, 3, a.stream);
    }
    if (!loss_done && !a.defer_loss_sum && launch_loss_sum(a, pl) != hipSuccess) return GC_ERR_HIP;
    prof_mark(call, 4, a.stream);
    if (g_prof.on) g_prof.calls++;
    return GC_OK;
  }
  if (a.both) {
    if (launch_stats_both(a, pl, *a.both) != hipSuccess) return GC_ERR_HIP;
  } else if (!a.lse2_t) {
    e = pl.route == ROUTE_MFMA ? launch_stats_mfma(a, pl) : pl.route == ROUTE_PLANES ? launch_stats_planes(a, pl) : launch_stats_generic(a, pl);
    if (e != hipSuccess) return GC_ERR_HIP;
  }
  prof_mark(call, 1, a.stream);
  if (a.both) {
    if (launch_both_merge(a, pl, *a.both) != hipSuccess) return GC_ERR_HIP;
  } else if (!a.lse2_t && !merges_itself(a, pl)) {
    e = launch_stats_merge(a, pl);
    if (e != hipSuccess) return GC_ERR_HIP;
  }
  prof_mark(call, 2, a.stream);
  if (a.dq || a.dp || a.dz) {
    e = pl.route == ROUTE_MFMA ? launch_grad_mfma(a, pl) : pl.route == ROUTE_PLANES ? launch_grad_planes(a, pl) : launch_grad_generic(a, pl);  // records mark 3 after its main kernel(s)
    if (e != hipSuccess) return GC_ERR_HIP;
  } else {
    prof_mark(call, 3, a.stream);
  }
  prof_mark(call, 4, a.stream);
  if (g_prof.on) g_prof.calls++;
  return GC_OK;
}

static int check_loss_args(int dt, const void* q, const void* p, const int32_t* pos_idx, int B, int P, int d,
                           float scale, float temp, unsigned flags) {
  if (!q || !p || !pos_idx) return GC_ERR_NULL;
  if (!shape_ok(B, P, d)) return GC_ERR_SHAPE;
  if (!(scale > 0.f) || !(temp > 0.f) || !std::isfinite(scale) || !std::isfinite(temp)) return GC_ERR_SHAPE;
  if (!std::isfinite(scale / temp) || !(scale / temp > 0.f)) return GC_ERR_SHAPE;
  if (dt != GC_F32 && dt != GC_BF16) return GC_ERR_UNSUPPORTED;
  if (flags & ~(GC_MASK_SELF | GC_PATH_ONLINE | GC_PATH_STATS_PASS | GC_CACHE_BF16)) return GC_ERR_UNSUPPORTED;
  if ((flags & GC_CACHE_BF16) && !(dt == GC_BF16 && d % 128 == 0 && d >= 128 && d <= 768)) return GC_ERR_UNSUPPORTED;
  if ((flags & GC_PATH_ONLINE) && (flags & GC_PATH_STATS_PASS)) return GC_ERR_UNSUPPORTED;
  if ((flags & GC_MASK_SELF) && (B != P || P < 2)) return GC_ERR_SHAPE;
  return GC_OK;
}

__global__ void pair_index_kernel(int32_t* r, int n, int* zero) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r[i] = i ^ 1;
  if (i == 0) *zero = 0;
}

// rinv[r[i]] = i; entries that no r[i] points at keep -1 (then r is no bijection, and the second direction of the
// symmetric loss reports them as positives out of range)
__global__ void fill_i32_kernel(int32_t* x, int n, int v, int* zero) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = v;
  if (i == 0) *zero = 0;
}
__global__ void invert_perm_kernel(const int32_t* r, int32_t* rinv, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const int j = r[i];
    if (j >= 0 && j < n) rinv[j] = i;
  }
}

}  // namespace gc

using namespace gc;

extern "C" {

const char* gc_strerror(int status) {
  switch (status) {
    case GC_OK: return "ok";
    case GC_ERR_NULL: return "a required pointer is NULL";
    case GC_ERR_SHAPE: return "invalid size, scale or temperature";
    case GC_ERR_UNSUPPORTED: return "unsupported dtype, flag or shape";
    case GC_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case GC_ERR_POS_IDX: return "pos_idx value outside [0, P)";
    case GC_ERR_HIP: return "HIP runtime call failed";
    case GC_ERR_TOO_LARGE: return "shape needs more scratch than the static buffer holds (GC_STATIC_SCRATCH_BYTES)";
    default: return "unknown gc_status";
  }
}

size_t gc_workspace_bytes(int B, int P, int d, int dt) {
  if (!shape_ok(B, P, d) || (dt != GC_F32 && dt != GC_BF16)) return 0;
  return make_loss_plan(B, P, d, (gc_dtype)dt, false).total;
}

static int loss_with_plan(const LossPlan& pl, gc_dtype dt, const void* q, const void* p, const int32_t* pos_idx, int B, int P, int d,
                          float scale, float temp, unsigned flags, float* loss, float* dq, float* dp, float* lse,
                          int32_t* argmax, void* workspace, void* stream) {
  LossArgs a{};
  a.dt = dt; a.q = q; a.p = p; a.pos_idx = pos_idx; a.B = B; a.P = P; a.d = d;
  a.alpha = scale / temp; a.flags = flags;
  a.loss = loss; a.dq = dq; a.dp = dp; a.lse = lse; a.argmax = argmax; a.dz = nullptr;
  a.ws = (char*)workspace; a.stream = (hipStream_t)stream;
  return run_loss(a, pl);
}

int gc_loss_and_rep_grad_ex(int dt_int, const void* q, const void* p, const int32_t* pos_idx, int B, int P, int d,
                            float scale, float temp, unsigned flags, float* loss, float* dq, float* dp, float* lse,
                            int32_t* argmax, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_loss_args(dt_int, q, p, pos_idx, B, P, d, scale, temp, flags);
  if (rc != GC_OK) return rc;
  const gc_dtype dt = (gc_dtype)dt_int;
  if (!workspace || ((uintptr_t)workspace & 255)) return GC_ERR_WORKSPACE;
  const LossPlan pl = make_loss_plan(B, P, d, dt, false, workspace_bytes);
  if (workspace_bytes < pl.total) return GC_ERR_WORKSPACE;
  return loss_with_plan(pl, dt, q, p, pos_idx, B, P, d, scale, temp, flags, loss, dq, dp, lse, argmax, workspace, stream);
}

static int simple_loss(gc_dtype dt, const void* q, const void* p, const int32_t* pos_idx, int B, int P, int d,
                       float scale, float temp, float* loss, float* dq, float* dp, void* stream) {
  int rc = check_loss_args(dt, q, p, pos_idx, B, P, d, scale, temp, 0);
  if (rc != GC_OK) return rc;
  if (!loss || !dq || !dp) return GC_ERR_NULL;
  LossPlan pl = make_loss_plan(B, P, d, dt, false);
  void* ws = nullptr;
  size_t have = 0;
  while ((rc = own_workspace(pl.total, (hipStream_t)stream, &ws, &have)) != GC_OK) {
    // a capture cannot grow the buffer: what fits the one there is?  A device without room: what needs less?
    const LossPlan less = make_loss_plan(B, P, d, dt, false, rc == GC_ERR_UNSUPPORTED ? have : pl.total - 1);
    if (less.total >= pl.total || (rc == GC_ERR_UNSUPPORTED && (!ws || less.total > have))) return rc;
    pl = less;
  }
  OwnCall call;
  rc = own_workspace_enter((hipStream_t)stream, call);
  if (rc != GC_OK) return rc;
  rc = loss_with_plan(pl, dt, q, p, pos_idx, B, P, d, scale, temp, 0, loss, dq, dp, nullptr, nullptr, ws, stream);
  const int rc2 = own_workspace_leave((hipStream_t)stream, call);   // also after a failed launch: some kernels may be queued
  return rc != GC_OK ? rc : rc2;
}

int gc_loss_and_rep_grad_bf16(const void* q, const void* p, const int32_t* pos_idx, int B, int P, int d, float scale,
                              float temp, float* loss, float* dq, float* dp, void* stream) {
  return simple_loss(GC_BF16, q, p, pos_idx, B, P, d, scale, temp, loss, dq, dp, stream);
}

int gc_loss_and_rep_grad_bf16_static(const void* q, const void* p, const int32_t* pos_idx, int B, int P, int d,
                                     float scale, float temp, float* loss, float* dq, float* dp, void* stream) {
  int rc = check_loss_args(GC_BF16, q, p, pos_idx, B, P, d, scale, temp, 0);
  if (rc != GC_OK) return rc;
  if (!loss || !dq || !dp) return GC_ERR_NULL;
  LossPlan pl = make_loss_plan(B, P, d, GC_BF16, false);
  if (!pl.use_mfma) pl = make_loss_plan(B, P, d, GC_BF16, false, (size_t)GC_STATIC_SCRATCH_BYTES);
  if (pl.total > (size_t)GC_STATIC_SCRATCH_BYTES) return GC_ERR_TOO_LARGE;
  if (pl.use_mfma) {
    struct Kept { int B, P, d; bool takes; };   // (the thread's last shape, as the plan's)
    static thread_local Kept kept{};
    if (kept.B != B || kept.P != P || kept.d != d) kept = Kept{B, P, d, static_takes(B, P, d)};
    if (!kept.takes) return GC_ERR_TOO_LARGE;
  }
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != GC_OK) return rc;
  // every word of the workspace that a kernel of this path reads has been written by an earlier kernel of the same
  // call (statistics, partial sums, the error word): nothing has to start at zero
  return loss_with_plan(pl, GC_BF16, q, p, pos_idx, B, P, d, scale, temp, 0, loss, dq, dp, nullptr, nullptr, ws, stream);
}

int gc_loss_and_rep_grad_f32(const float* q, const float* p, const int32_t* pos_idx, int B, int P, int d, float scale,
                             float temp, float* loss, float* dq, float* dp, void* stream) {
  return simple_loss(GC_F32, q, p, pos_idx, B, P, d, scale, temp, loss, dq, dp, stream);
}

int gc_check_async_error(const void* workspace) {
  const void* ws[2] = {workspace, nullptr};
  int word = 0;
  if (!workspace) {   // the library's own buffers of this device, as far as they have been used
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return GC_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_ws_mutex);
    ws[0] = g_ws_ptr[dev];
    ws[1] = g_scratch_ptr[dev];
    // what a replayed graph has left in a buffer that only it uses is reported once
    for (int i = 0; i < g_ws_nkept[dev]; i++) {
      if (hipMemcpy(&word, g_ws_kept[dev][i], sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) return GC_ERR_HIP;
      if (!word) continue;
      word = 0;
      if (hipMemcpy(g_ws_kept[dev][i], &word, sizeof(int), hipMemcpyHostToDevice) != hipSuccess) return GC_ERR_HIP;
      return GC_ERR_POS_IDX;
    }
  }
  for (const void* w : ws) {
    if (!w) continue;
    if (hipMemcpy(&word, w, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) return GC_ERR_HIP;
    if (word) return GC_ERR_POS_IDX;
  }
  return GC_OK;
}

int gc_profile_begin(int max_calls) {
  if (max_calls < 1 || max_calls > (1 << 16)) return GC_ERR_SHAPE;
  if (g_prof.ev) return GC_ERR_UNSUPPORTED;  // already open
  g_prof.ev = new hipEvent_t[(size_t)max_calls * kMarks];
  for (int i = 0; i < max_calls * kMarks; i++)
    if (hipEventCreate(&g_prof.ev[i]) != hipSuccess) {   // give back what was made: a later begin starts afresh
      for (int k = 0; k < i; k++) (void)hipEventDestroy(g_prof.ev[k]);
      delete[] g_prof.ev;
      g_prof.ev = nullptr;
      return GC_ERR_HIP;
    }
  g_prof.max_calls = max_calls;
  g_prof.calls = 0;
  g_prof.on = true;
  return GC_OK;
}

int gc_profile_end(float* ms_stats, float* ms_merge, float* ms_grad, float* ms_reduce, int* calls) {
  if (!g_prof.ev) return GC_ERR_UNSUPPORTED;
  g_prof.on = false;
  const int n = g_prof.calls < g_prof.max_calls ? g_prof.calls : g_prof.max_calls;
  double acc[4] = {0, 0, 0, 0};
  int rc = GC_OK;
  for (int c = 0; c < n && rc == GC_OK; c++) {
    if (hipEventSynchronize(g_prof.ev[c * kMarks + 4]) != hipSuccess) { rc = GC_ERR_HIP; break; }
    for (int k = 0; k < 4; k++) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, g_prof.ev[c * kMarks + k], g_prof.ev[c * kMarks + k + 1]) != hipSuccess) rc = GC_ERR_HIP;
      acc[k] += ms;
    }
  }
  for (int i = 0; i < g_prof.max_calls * kMarks; i++) (void)hipEventDestroy(g_prof.ev[i]);
  delete[] g_prof.ev;
  g_prof.ev = nullptr;
  if (rc != GC_OK) return rc;
  if (ms_stats) *ms_stats = n ? (float)(acc[0] / n) : 0.f;
  if (ms_merge) *ms_merge = n ? (float)(acc[1] / n) : 0.f;
  if (ms_grad) *ms_grad = n ? (float)(acc[2] / n) : 0.f;
  if (ms_reduce) *ms_reduce = n ? (float)(acc[3] / n) : 0.f;
  if (calls) *calls = n;
  g_prof.max_calls = g_prof.calls = 0;
  return GC_OK;
}

size_t gc_ntxent_workspace_bytes(int n_views, int d) {
  if (n_views < 2 || (n_views & 1) || !shape_ok(n_views, n_views, d)) return 0;
  return make_loss_plan(n_views, n_views, d, GC_BF16, true).total;
}

int gc_ntxent_loss_and_grad_bf16(const void* z, int n_views, int d, float temp, float* loss, float* dz,
                                 void* workspace, size_t workspace_bytes, void* stream) {
  if (!z) return GC_ERR_NULL;
  if (n_views < 2 || (n_views & 1) || !shape_ok(n_views, n_views, d)) return GC_ERR_SHAPE;
  if (!(temp > 0.f) || !std::isfinite(temp) || !std::isfinite(1.f / temp)) return GC_ERR_SHAPE;
  if (!workspace || ((uintptr_t)workspace & 255)) return GC_ERR_WORKSPACE;
  const LossPlan pl = make_loss_plan(n_views, n_views, d, GC_BF16, true, workspace_bytes);
  if (workspace_bytes < pl.total) return GC_ERR_WORKSPACE;
  LossArgs a{};
  a.dt = GC_BF16; a.q = z; a.p = z; a.B = n_views; a.P = n_views; a.d = d;
  a.alpha = 1.f / temp; a.flags = GC_MASK_SELF;
  a.loss = loss; a.dz = dz;
  a.ws = (char*)workspace; a.stream = (hipStream_t)stream;
  int32_t* r = (int32_t*)(a.ws + pl.off_pos_idx);
  a.wide = (int*)(a.ws + pl.off_err) + 2;
  if (pl.one_walk) a.wexp = (float*)(a.ws + pl.off_part_idx);
  const BothPlan both = plan_both(n_views, d, true, pl);
  if (both.use) {   // the pairs are written by the kernel that merges the statistics
    a.both = &both;
    a.pos_idx = (const int32_t*)(a.ws + pl.off_pos_pad);
  } else {
    pair_index_kernel<<<(n_views + 255) / 256, 256, 0, a.stream>>>(r, n_views, a.wide);
    if (hipGetLastError() != hipSuccess) return GC_ERR_HIP;
    a.pos_idx = r;
  }
  return run_loss(a, pl);
}

// Workspace of the symmetric loss: [loss workspace, direction 1][direction 2][r^-1][two losses][4 gradient buffers].
// With the MFMA kernels one gradient pass serves both directions: the second workspace then holds statistics only
// and there are no gradient buffers.  The general widths share the packed inputs and partials between the directions.
struct SymPlan { LossPlan pl; size_t off2, off_rinv, off_l, off_g, total; };
static SymPlan sym_plan_of(const LossPlan& pl, int n, int d) {
  SymPlan sp{};
  sp.pl = pl;
  size_t off = align_up(sp.pl.total, 256);
  sp.off2 = off; off = align_up(off + (sp.pl.route == ROUTE_GENERAL ? sp.pl.total : sp.pl.off_dq_part), 256);
  sp.off_rinv = off; off = align_up(off + (size_t)n * 4, 256);
  sp.off_l = off; off += 256;
  sp.off_g = off; off += sp.pl.use_mfma ? 0 : 4 * align_up((size_t)n * d * 4, 256);
  sp.total = off;
  return sp;
}
static SymPlan make_sym_plan(int n, int d, size_t limit = (size_t)-1) {
  const SymPlan sp = sym_plan_of(make_loss_plan(n, n, d, GC_BF16, false), n, d);
  if (sp.total <= limit) return sp;
  return sym_plan_of(choose_plan(n, n, d, GC_BF16, false, [=](const LossPlan& pl) { return sym_plan_of(pl, n, d).total <= limit; }), n, d);
}

size_t gc_bidirectional_workspace_bytes(int n, int d) {
  if (n < 1 || !shape_ok(n, n, d)) return 0;
  return make_sym_plan(n, d).total;
}

int gc_bidirectional_loss_and_rep_grad_bf16(const void* q, const void* p, const int32_t* pos_idx, int n, int d, float scale,
                                            float temp, float* loss, float* dq, float* dp, void* workspace,
                                            size_t workspace_bytes, void* stream) {
  int rc = check_loss_args(GC_BF16, q, p, pos_idx, n, n, d, scale, temp, 0);
  if (rc != GC_OK) return rc;
  if (!loss || !dq || !dp) return GC_ERR_NULL;
  if (!workspace || ((uintptr_t)workspace & 255)) return GC_ERR_WORKSPACE;
  const SymPlan sp = make_sym_plan(n, d, workspace_bytes);
  if (workspace_bytes < sp.total) return GC_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  hipStream_t s = (hipStream_t)stream;
  int32_t* rinv = (int32_t*)(ws + sp.off_rinv);
  float* l = (float*)(ws + sp.off_l);
  int* wide = (int*)(ws + sp.pl.off_err) + 2;
  const BothPlan both = sp.pl.use_mfma ? plan_both(n, d, false, sp.pl) : BothPlan{};
  if (!both.use) {   // (else the statistics pass inverts the pairing, and its merge checks it)
    fill_i32_kernel<<<(n + 255) / 256, 256, 0, s>>>(rinv, n, -1, wide);
    invert_perm_kernel<<<(n + 255) / 256, 256, 0, s>>>(pos_idx, rinv, n);
    if (hipGetLastError() != hipSuccess) return GC_ERR_HIP;
  }
  LossArgs a{};
  a.dt = GC_BF16; a.B = n; a.P = n; a.d = d; a.alpha = scale / temp; a.stream = s;
  a.defer_loss_sum = true;   // one launch sums the row losses of both directions at the end
  LossArgs a1, a2;
  if (sp.pl.use_mfma) {
    a.wide = wide;
    a1 = a2 = a;   // (for the sum of the row losses)
    a1.q = q; a1.p = p; a1.pos_idx = pos_idx; a1.loss = l; a1.ws = ws; a1.wexp = (float*)(ws + sp.pl.off_part_idx);
    a2.q = p; a2.p = q; a2.pos_idx = rinv; a2.loss = l + 1; a2.ws = ws + sp.off2; a2.wexp = (float*)(ws + sp.off2 + sp.pl.off_part_idx);
    if (!both.use) {   // statistics of both directions (Eq. 1 as it stands, then with the two sides exchanged) ...
      rc = run_loss(a1, sp.pl);
      if (rc != GC_OK) return rc;
      rc = run_loss(a2, sp.pl);
      if (rc != GC_OK) return rc;
    }
    // ... and one gradient pass with the mean of the two softmaxes as coefficients
    a.q = q; a.p = p; a.pos_idx = pos_idx; a.loss = nullptr; a.ws = ws; a.dq = dq; a.dp = dp;
    a.lse2_t = (const float*)(ws + sp.off2 + sp.pl.off_lse2);
    a.wexp = a1.wexp; a.wexp_t = a2.wexp;
    if (both.use) { a.both = &both; a.ws_t = ws + sp.off2; }   // ... (the statistics in one pass where that is faster)
    a.pos_inv = rinv;
    a.sym[0] = &a1; a.sym[1] = &a2; a.sym_loss = loss;
    a.zero_word = (const int*)(ws + sp.pl.off_err) + 1;   // zeroed by the first direction's merge, raised by nobody here
    return run_loss(a, sp.pl);   // (its last launch also sums the row losses)
  } else {
    const size_t gsz = align_up((size_t)n * d * 4, 256);
    float* g[4];
    for (int i = 0; i < 4; i++) g[i] = (float*)(ws + sp.off_g + i * gsz);
    a.grad_mul = 0.5f;
    // direction 1: anchors against targets (Eq. 1); direction 2: the same with the two sides exchanged
    a.q = q; a.p = p; a.pos_idx = pos_idx; a.loss = l; a.dq = g[0]; a.dp = g[1]; a.ws = ws;
    a1 = a;
    rc = run_loss(a, sp.pl);
    if (rc != GC_OK) return rc;
    a.q = p; a.p = q; a.pos_idx = rinv; a.loss = l + 1; a.dq = g[2]; a.dp = g[3]; a.ws = ws + sp.off2;
    a.ws2 = ws;   // its statistics are its own (the row losses of both are summed at the end), the rest is free again
    a2 = a;
    rc = run_loss(a, sp.pl);
    if (rc != GC_OK) return rc;
    // dL/df = Eq. 5 of direction 1 + Eq. 6 of direction 2, dL/dg the other two; fixed order
    const size_t ne = (size_t)n * d;
    ReduceJob j[2] = {};
    j[0].out = dq; j[0].ptr[0] = g[0]; j[0].ptr[1] = g[3];
    j[1].out = dp; j[1].ptr[0] = g[1]; j[1].ptr[1] = g[2];
    for (ReduceJob& k : j) { k.n = ne; k.nsrc = 2; k.count[0] = k.count[1] = 1; }
    if (launch_reduce_jobs(j, 2, s) != hipSuccess) return GC_ERR_HIP;
  }
  return launch_sym_loss_sum(a1, a2, sp.pl, loss) == hipSuccess ? GC_OK : GC_ERR_HIP;
}

}  // extern "C"
