// FP64 pivoted Jacobi phase (Algorithm 1, greedy or gap-aware pivots of eq. (1)) of one
// large matrix on several workgroups at once.
//
// The arithmetic, the pivot rule, the per-row caches of Sec. 3.2 and the mirrored storage
// of A are those of the one-workgroup kernels (jacobi_wg.h); only the reductions are
// spread out.  G workgroups own the rows k = T + i G 64 (T = 64 g + lane, i < RM).  Three
// kernels:
//   k_jacobi_spec4     several rotations per exchange, four waves per workgroup, one row per
//                      lane (n <= 4096);
//   k_jacobi_spec_mw   the same on one wave per workgroup, two rows per lane (n > 4096): the
//                      loop of jacobi_spec.h;
//   k_jacobi_mw        one rotation per exchange, one wave per workgroup, for the stop rules
//                      that need more than the best pivot after each rotation.
// The last of them, every rotation:
//   1. each wave reduces its own candidates (best cached pivot over its rows, best entries
//      of the new rows p and q of the last rotation) and publishes them in a slot of a
//      double-buffered exchange area;
//   2. it arrives at a counter barrier, and when all G have arrived it reads all G slots
//      and reduces them the same way, so every workgroup holds the same winner;
//   3. each workgroup applies the rotation to its own rows (rows p, q of A at its columns,
//      and the mirrored columns p, q of its rows), refreshes its caches and computes its
//      candidates for the next round.
// A full rescan of a stale row is one more exchange round.
//
// Placement and memory ordering: workgroups are dispatched to the XCDs round-robin, so the
// grid is 8 G and only workgroups with blockIdx % 8 == 0 work; they share XCD 0 and its
// L2.  Loads of A and of the exchange area are relaxed agent-scope atomics (they miss the
// per-CU cache and read L2), stores are workgroup-scope (acknowledged by that L2), and a
// wave waits for its stores to be acknowledged before it arrives at a barrier.  Where a
// round's stores may meet other workgroups' loads of the same round (entries between two of
// its pivots' rows), the vote on the proven rotations comes between them: a workgroup votes
// after its loads have returned and stores after all have voted.  A start barrier checks
// every workgroup's XCC id: if they do not share one XCD (or a start wait runs out) the
// kernel returns without touching the state and the host runs the one-workgroup kernel
// instead.  Every wait is bounded; a wait that runs out sets an abort flag that ends all
// workgroups.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"
#include "jacobi_device.h"
#include "jacobi_spec.h"
#include "kernels.h"
#include "mw_exchange.h"

namespace je {

constexpr int kMwWords = 28;            // words of one workgroup's slot: 6 candidates x 4 + 3 sums

// A candidate as four words of a slot: score, value, bound, and (row | flag << 31,
// column) as two 32-bit halves (row and column are non-negative ints).
__device__ __forceinline__ void put_cand(double* w, const Cand& x) {
  st_ag(w + 0, x.s);
  st_ag(w + 1, x.a);
  st_ag(w + 2, x.u);
  const unsigned lo = (unsigned)x.i | ((unsigned)(x.f & 1) << 31);
  const long long pk = (long long)lo | ((long long)(unsigned)x.c << 32);
  st_ag(w + 3, __longlong_as_double(pk));
}

__device__ __forceinline__ Cand get_cand(const double* w) {
  Cand x;
  x.s = ld_ag(w + 0);
  x.a = ld_ag(w + 1);
  x.u = ld_ag(w + 2);
  const unsigned long long pk = (unsigned long long)__double_as_longlong(ld_ag(w + 3));
  const unsigned lo = (unsigned)(pk & 0xffffffffull);
  x.i = (int)(lo & 0x7fffffffu);
  x.f = (int)(lo >> 31);
  x.c = (int)(unsigned)(pk >> 32);
  x.pad = 0;
  return x;
}

template <int RM, bool GAP>
__global__ __launch_bounds__(64) void k_jacobi_mw(JDesc d, long long log_base, MwCtl* mc,
                                                  double* xb, int G) {
  if (blockIdx.x % kMwStride) return;
  const int g = blockIdx.x / kMwStride;
  if (g >= G) return;
  extern __shared__ double s_diag[];
  const int lane = threadIdx.x;
  const int T = g * kWave + lane, GT = G * kWave;
  const int n = d.n;
  const bool use_cert = !GAP && d.stop == STOP_CERT;
  const bool use_off = d.stop == STOP_OFF;
  const int ld = d.ld;
  double* gA = d.A;
  auto ld_a = [&](int r, int c) -> double { return ld_ag(gA + (size_t)r * ld + c); };
  auto st_a = [&](int r, int c, double v) { st_ag(gA + (size_t)r * ld + c, v); };

  int round = 1;
  if (!mw_start(mc, G, g, round)) return;

  // ---- per-thread rows k = T + i GT; the whole diagonal in LDS
  double dk[RM], bs[RM], bv[RM], bu[RM], cb[RM], cu[RM], of2[RM];
  int ba[RM], bst[RM], ca[RM], cst[RM], tk[RM];
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    int k = T + i * GT;
    if (k < n) {
      dk[i] = d.diag[k]; bs[i] = d.bs[k]; ba[i] = d.ba[k]; bv[i] = d.bv[k]; bst[i] = d.bst[k];
      bu[i] = d.bu[k]; of2[i] = d.off2[k]; tk[i] = d.ts[k];
      if (use_cert) { cb[i] = d.cb[k]; ca[i] = d.ca[k]; cst[i] = d.cst[k]; cu[i] = d.cu[k]; }
      else { cb[i] = -1.0; ca[i] = -1; cst[i] = 0; cu[i] = -1.0; }
    } else {
      dk[i] = 0.0; bs[i] = -1.0; ba[i] = -1; bv[i] = 0.0; bst[i] = 0; bu[i] = -1.0; of2[i] = 0.0;
      tk[i] = 0; cb[i] = -1.0; ca[i] = -1; cst[i] = 0; cu[i] = -1.0;
    }
  }
  for (int l = lane; l < n; l += kWave) s_diag[l] = d.diag[l];
  __syncthreads();

  long long rot = d.ctl->rotations;
  long long rescans = 0;
  int status = ST_OK, done = 0, failed = 0;
  const double thr = d.thr;
  int lp = -1, lq = -1, lrot = 0;
  double lapp = 0.0, laqq = 0.0;
  bool pend = false;
  Cand rp = empty_cand(), rq = rp, cp = rp, cq = rp;
  double op = 0.0, oq = 0.0;
  Cand W = empty_cand(), C = empty_cand();
  double off_tot = 0.0;

  auto diag_of = [&](int x) -> double { return x == lp ? lapp : (x == lq ? laqq : s_diag[x]); };
  auto slot = [&](int b, int wg) -> double* { return xb + (size_t)(b * G + wg) * kMwWords; };
  // optional phase timers of workgroup 0 (10 ns ticks): local reductions, publishing and
  // the store acknowledgements, the barrier wait, reading and reducing the slots, the
  // rotation parameters with the row loads, the update
  const bool prof = d.prof != nullptr && g == 0;
  long long tph[6] = {0, 0, 0, 0, 0, 0}, tmark = 0;
  auto tick = [&]() -> long long { return prof ? (long long)wall_clock64() : 0; };
  auto lap = [&](int k) {
    if (prof) { const long long t = tick(); tph[k] += t - tmark; tmark = t; }
  };

  // Full rescan of row r's selection (which == 0) or certificate (which == 1) cache: each
  // workgroup scans its columns, one exchange round combines them.
  auto rescan = [&](int r, int which) -> bool {
    const double arr = diag_of(r);
    double vals[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int l = T + i * GT;
      vals[i] = (l < n && l != r) ? ld_a(r, l) : 0.0;
    }
    Cand x = empty_cand();
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int l = T + i * GT;
      if (l >= n || l == r) continue;
      double v = vals[i];
      double sc = which == 0 ? sel_score<GAP>(arr, dk[i], v) : gap_score(arr, dk[i], v);
      cand_top2(x, sc, l, v);
    }
    Cand e1 = empty_cand(), e2 = empty_cand();
    wave_best3(e1, 0, x, x.c, e2, 0);
    ++round;
    const int b = round & 1;
    if (lane == 0) put_cand(slot(b, g), x);
    if (!mw_sync(mc, G, round)) return false;
    Cand y = lane < G ? get_cand(slot(b, lane)) : empty_cand();
    Cand f1 = empty_cand(), f2 = empty_cand();
    wave_best3(f1, 0, y, y.c, f2, 0);
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      if (T + i * GT == r) {
        if (which == 0) { bs[i] = y.s; ba[i] = y.c; bv[i] = y.a; bu[i] = y.u; bst[i] = 0; }
        else { cb[i] = y.s; ca[i] = y.c; cu[i] = y.u; cst[i] = 0; }
      }
    }
    ++rescans;
    return true;
  };

  for (;;) {
    tmark = tick();
    // ---- per-thread candidates over own rows
    Cand x1 = empty_cand(), x4 = empty_cand();
    double o7 = 0.0;
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int k = T + i * GT;
      if (k >= n) continue;
      if (pend && (k == lp || k == lq)) continue;
      if (bs[i] > x1.s) { x1.s = bs[i]; x1.i = k; x1.c = ba[i]; x1.a = bv[i]; x1.f = bst[i]; }
      if (use_cert && cb[i] > x4.s) { x4.s = cb[i]; x4.i = k; x4.c = ca[i]; x4.f = cst[i]; }
      if (use_off) o7 += of2[i];
    }
    // ---- wave reductions (rp, rq, cp, cq are empty unless a rotation is pending)
    Cand w1 = x1, w2 = rp, w3 = rq, w4 = x4, w5 = cp, w6 = cq;
    wave_best3(w1, x1.i, w2, rp.c, w3, rq.c);
    if (use_cert) wave_best3(w4, x4.i, w5, cp.c, w6, cq.c);
    double s7 = 0.0, s8 = 0.0, s9 = 0.0;
    if (use_off) { s7 = wave_sum_fast(o7); s8 = wave_sum_fast(op); s9 = wave_sum_fast(oq); }
    lap(0);
    // ---- exchange: publish, wait for all, read all
    ++round;
    const int b = round & 1;
    {
      double* my = slot(b, g);
      if (lane == 0) put_cand(my, w1);
      if (lane == 1) put_cand(my + 4, w2);
      if (lane == 2) put_cand(my + 8, w3);
      if (use_cert) {
        if (lane == 3) put_cand(my + 12, w4);
        if (lane == 4) put_cand(my + 16, w5);
        if (lane == 5) put_cand(my + 20, w6);
      }
      if (use_off && lane == 6) { st_ag(my + 24, s7); st_ag(my + 25, s8); st_ag(my + 26, s9); }
    }
    if (prof) { __builtin_amdgcn_s_waitcnt(0); lap(1); }
    if (!mw_sync(mc, G, round)) { failed = 1; break; }
    lap(2);
    {
      const double* sl = slot(b, lane < G ? lane : 0);
      Cand y1 = empty_cand(), y2 = y1, y3 = y1;
      if (lane < G) { y1 = get_cand(sl); y2 = get_cand(sl + 4); y3 = get_cand(sl + 8); }
      wave_best3(y1, y1.i, y2, y2.c, y3, y3.c);
      w1 = y1; w2 = y2; w3 = y3;
      if (use_cert) {
        Cand y4 = empty_cand(), y5 = y4, y6 = y4;
        if (lane < G) { y4 = get_cand(sl + 12); y5 = get_cand(sl + 16); y6 = get_cand(sl + 20); }
        wave_best3(y4, y4.i, y5, y5.c, y6, y6.c);
        w4 = y4; w5 = y5; w6 = y6;
      }
      if (use_off) {
        // fixed order over the workgroups: the same sums in every workgroup
        double a7 = 0.0, a8 = 0.0, a9 = 0.0;
        for (int x = 0; x < G; ++x) {
          const double* sx = slot(b, x);
          a7 += ld_ag(sx + 24); a8 += ld_ag(sx + 25); a9 += ld_ag(sx + 26);
        }
        s7 = a7; s8 = a8; s9 = a9;
      }
    }
    lap(3);
    // ---- fold in the rows of the last rotation
    W = w1;
    C = w4;
    off_tot = s7;
    if (pend) {
      if (better(w2.s, lp, W.s, W.i)) W = Cand{w2.s, w2.a, w2.u, lp, w2.c, 0, 0};
      if (better(w3.s, lq, W.s, W.i)) W = Cand{w3.s, w3.a, w3.u, lq, w3.c, 0, 0};
      if (use_cert) {
        if (better(w5.s, lp, C.s, C.i)) C = Cand{w5.s, 0.0, w5.u, lp, w5.c, 0, 0};
        if (better(w6.s, lq, C.s, C.i)) C = Cand{w6.s, 0.0, w6.u, lq, w6.c, 0, 0};
      }
      off_tot = (s7 + s8) + s9;
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        int k = T + i * GT;
        if (k == lp) {
          bs[i] = w2.s; ba[i] = w2.c; bv[i] = w2.a; bu[i] = w2.u; bst[i] = 0; of2[i] = s8;
          if (use_cert) { cb[i] = w5.s; ca[i] = w5.c; cu[i] = w5.u; cst[i] = 0; }
        } else if (k == lq) {
          bs[i] = w3.s; ba[i] = w3.c; bv[i] = w3.a; bu[i] = w3.u; bst[i] = 0; of2[i] = s9;
          if (use_cert) { cb[i] = w6.s; ca[i] = w6.c; cu[i] = w6.u; cst[i] = 0; }
        }
      }
      if (lane == 0) { s_diag[lp] = lapp; s_diag[lq] = laqq; }
      pend = false;
      rp = empty_cand(); rq = rp; cp = rp; cq = rp;
      op = 0.0; oq = 0.0;
    }
    if (n < 2) { done = 1; break; }
    // ---- the winner must be exact
    if (W.f) {
      if (!rescan(W.i, 0)) { failed = 1; break; }
      continue;
    }
    // ---- stop rules (checked before every rotation)
    if (d.stop == STOP_CERT) {
      if (GAP) {
        if (W.s <= thr) { done = 1; break; }
      } else {
        if (C.s <= thr) { done = 1; break; }
        if (C.f) {
          if (!rescan(C.i, 1)) { failed = 1; break; }
          continue;
        }
      }
    } else if (d.stop == STOP_OFF) {
      if (sqrt(off_tot) <= thr) { done = 1; break; }
    } else {
      if (W.s <= thr) { done = 1; break; }
    }
    if (rot >= d.maxrot) { status = ST_MAXROT; done = 1; break; }
    if (W.a == 0.0) { status = ST_STALL; done = 1; break; }
    if (rot - log_base >= d.log_cap) break;  // log full: drain and resume

    // ---- rotation (p, q): issue the row loads first, the parameters overlap them
    const int p = min(W.i, W.c), q = max(W.i, W.c);
    double xv[RM], yv[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int k = T + i * GT;
      xv[i] = 0.0; yv[i] = 0.0;
      if (k >= n || k == p || k == q) continue;
      xv[i] = ld_a(p, k);
      yv[i] = ld_a(q, k);
    }
    const double apq = W.a;
    const double app = diag_of(p), aqq = diag_of(q);
    double t, c, s;
    rot_params<double>(app, aqq, apq, t, c, s);
    const double napp = app + t * apq;
    const double naqq = aqq - t * apq;
    const int nts = (int)(rot + 1);
    if (prof) { __builtin_amdgcn_s_waitcnt(0); lap(4); }
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int k = T + i * GT;
      if (k >= n) continue;
      if (k == p) {
        st_a(q, p, 0.0);
        st_a(p, q, 0.0);
        dk[i] = napp; tk[i] = nts;
        cand_top2(rq, 0.0, p, 0.0);
        if (use_cert) cand_top2(cq, 0.0, p, 0.0);
        continue;
      }
      if (k == q) {
        dk[i] = naqq; tk[i] = nts;
        cand_top2(rp, 0.0, q, 0.0);
        if (use_cert) cand_top2(cp, 0.0, q, 0.0);
        continue;
      }
      const double x = xv[i], y = yv[i];
      const double xn = c * x + s * y;
      const double yn = c * y - s * x;
      st_a(p, k, xn);
      st_a(q, k, yn);
      st_a(k, p, xn);
      st_a(k, q, yn);
      const double sp = sel_score<GAP>(dk[i], napp, xn);
      const double sq = sel_score<GAP>(dk[i], naqq, yn);
      refresh_entry(bs[i], ba[i], bv[i], bu[i], bst[i], p, q, sp, xn, sq, yn);
      cand_top2(rp, sp, k, xn);
      cand_top2(rq, sq, k, yn);
      if (use_cert) {
        const double lpv = gap_score(dk[i], napp, xn);
        const double lqv = gap_score(dk[i], naqq, yn);
        double dummy = 0.0;
        refresh_entry(cb[i], ca[i], dummy, cu[i], cst[i], p, q, lpv, 0.0, lqv, 0.0);
        cand_top2(cp, lpv, k, 0.0);
        cand_top2(cq, lqv, k, 0.0);
      }
      if (use_off) { op += xn * xn; oq += yn * yn; }
    }
    if (g == 0 && lane == 0) d.log[rot - log_base] = RotEntry{p, q, c, s};
    lap(5);
    lp = p; lq = q; lapp = napp; laqq = naqq; lrot = nts;
    pend = true;
    ++rot;
  }
  if (failed) return;  // the host reports a device error; the state is not resumable

  // ---- write the state back (a later launch may resume from it)
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    int k = T + i * GT;
    if (k < n) {
      d.diag[k] = dk[i]; d.bs[k] = bs[i]; d.ba[k] = ba[i]; d.bv[k] = bv[i]; d.bst[k] = bst[i];
      d.bu[k] = bu[i]; d.off2[k] = of2[i]; d.ts[k] = tk[i];
      if (use_cert) { d.cb[k] = cb[i]; d.ca[k] = ca[i]; d.cst[k] = cst[i]; d.cu[k] = cu[i]; }
    }
  }
  if (prof && lane == 0)
    for (int k = 0; k < 6; ++k) d.prof[k] += tph[k];
  if (g == 0 && lane == 0) {
    JCtl* ctl = d.ctl;
    ctl->rotations = rot;
    ctl->rescans += rescans;
    ctl->status = status;
    ctl->done = done;
    ctl->final_sel = W.s;
    ctl->final_cert = GAP ? W.s : C.s;
    ctl->final_off = sqrt(off_tot);
  }
}

// ------------------------------------------------------------------ speculative rounds
// The exchange of the speculative loop (jacobi_spec.h) between G one-wave workgroups.  A
// round costs two waits: one on the slots of candidates (publishing, store acknowledgements,
// counter barrier, slot read), one on the vote.  The vote is a single 64-bit atomic per
// workgroup, which carries the arrival and the first stage it could not prove: arrivals in
// the low byte, seven bits per stage above it (at most 64 workgroups each).
struct MwExchange {
  static constexpr bool kExchange = true;
  static constexpr int kSlotWords = 2 * kMwMaxGroups * 4 * 4;  // two rounds, four a workgroup
  MwCtl* mc;
  double* xb;
  double* A;
  double* s_diag;
  int G, g, T, GT, ld_, lane, round, votes;
  bool alive;

  __device__ __forceinline__ bool first_wave() const { return g == 0; }
  __device__ __forceinline__ bool ok() const { return alive; }
  __device__ __forceinline__ double* slot(int b, int idx) const {
    return xb + (size_t)(b * kMwMaxGroups * 4 + idx) * 4;
  }
  __device__ __forceinline__ void publish(bool win, const SCand& x) {
    if (win) {
      double* p = slot((round + 1) & 1, 4 * g + (lane >> 4));
      st_ag(p, x.s);
      st_ag(p + 1, x.a);
      st_ag(p + 2, __longlong_as_double((long long)x.rc));
    }
  }
  __device__ __forceinline__ SCand gather(const SCand&) {
    ++round;
    alive = mw_sync(mc, G, round);
    SCand y = empty_scand();
    if (!alive) return y;
    SCand z[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      z[u] = empty_scand();
      if (u * 16 < G && lane + 64 * u < 4 * G) {
        const double* p = slot(round & 1, lane + 64 * u);
        z[u].s = ld_ag(p);
        z[u].a = ld_ag(p + 1);
        z[u].rc = (int)__double_as_longlong(ld_ag(p + 2));
      }
    }
    int yk = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int zk = scand_key(z[u].rc);
      if (z[u].s >= 0.0 && better(z[u].s, zk, y.s, yk)) { y = z[u]; yk = zk; }
    }
    return y;
  }
  // Words of the vote are used in turn; the word two votes ahead, which every workgroup has
  // left, is cleared here and acknowledged before the next candidates' barrier.
  __device__ __forceinline__ int vote(int F, int kk) {
    if (kk == 1) return 1;
    // the loads of this round are complete: after the vote other workgroups store into the
    // rows they came from
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    unsigned long long* word = &mc->vote[votes & 3];
    if (lane == 0) {
      unsigned long long add = 1;
      if (F < kk) add |= 1ull << (8 + 7 * (F - 1));
      __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    unsigned long long v = 0;
    int spins = 0;
    for (;;) {
      v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((int)(v & 0xff) >= G) break;
      if (++spins > kMwSpinLimit || (!(spins & 63) && ld_ag_i(&mc->abort))) {
        if (lane == 0) st_ag_i(&mc->abort, 1);
        alive = false;
        return 0;
      }
    }
    if (g == 0 && lane == 0)
      __hip_atomic_store(&mc->vote[(votes + 2) & 3], 0ull, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    ++votes;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    const unsigned long long fails = v >> 8;
    return __builtin_amdgcn_readfirstlane(fails ? (__ffsll((long long)fails) - 1) / 7 + 1 : kk);
  }
  __device__ __forceinline__ Cand best(const Cand& x) {
    ++round;
    double* my = xb + kSlotWords + (size_t)((round & 1) * G + g) * 4;
    if (lane == 0) put_cand(my, x);
    alive = mw_sync(mc, G, round);
    Cand y = empty_cand();
    if (!alive) return y;
    if (lane < G)
      y = get_cand(xb + kSlotWords + (size_t)((round & 1) * G + lane) * 4);
    Cand e1 = empty_cand(), e2 = empty_cand();
    wave_best3(e1, 0, y, y.c, e2, 0);
    return y;
  }
  __device__ __forceinline__ double ld(int r, int k, int) const {
    return ld_ag(A + (size_t)r * ld_ + k);
  }
  __device__ __forceinline__ double ld2(int r, int l) const { return ld_ag(A + (size_t)r * ld_ + l); }
  __device__ __forceinline__ void st(int r, int k, double v) { st_ag(A + (size_t)r * ld_ + k, v); }
  __device__ __forceinline__ void stm(int k, int r, double v) { st_ag(A + (size_t)k * ld_ + r, v); }
  __device__ __forceinline__ double diag(int k) const { return s_diag[k]; }
  __device__ __forceinline__ void set_diag(int p, int q, double dp, double dq, int) {
    s_diag[p] = dp;
    s_diag[q] = dq;
  }
};

template <int RM, int K, bool GAP>
__global__ __launch_bounds__(64) void k_jacobi_spec_mw(JDesc d, long long log_base, MwCtl* mc,
                                                       double* xb, int G) {
  if (blockIdx.x % kMwStride) return;
  const int g = blockIdx.x / kMwStride;
  if (g >= G) return;
  extern __shared__ double s_diag[];
  const int lane = threadIdx.x;
  int round = 1;
  if (!mw_start(mc, G, g, round)) return;
  for (int l = lane; l < d.n; l += kWave) s_diag[l] = d.diag[l];
  __syncthreads();
  MwExchange ex{mc, xb, d.A, s_diag, G, g, g * kWave + lane, G * kWave, d.ld, lane,
                     round, 0, true};
  spec_loop<RM, K, GAP>(d, log_base, ex);
}

// ------------------------------------------------------------------ speculative rounds, four
// waves per workgroup
// One row per lane (n <= 4096): the stages of a round are independent of each other up to the
// proof (the entries of a row that an earlier stage rotates are formed from that rotation's
// parameters), so the four waves of a workgroup hold the same 64 rows and take the stages j mod
// 4 each: the loads, new entries, scores and stores of a round spread over the CU's four SIMDs.
// Scores and entries meet in LDS; the selection, the proof and the caches, short and serial, are
// repeated by every wave on its own copy.  The exchanges use flags instead of counters: a
// workgroup stores its round number (with its vote) in a word of its own and all waves poll the
// G words with one load, 0.1 us a try against 0.4 us for the round trip of an atomic.
// The bound is the chain of short dependent steps of a round (about 2.9 rotations at n = 1024: per
// rotation 0.55 us selection and loads, 0.24 entries and scores, 0.15 proof, 0.19 vote, 0.2 stores
// and caches, 0.2 exchange).  Measured, FP64 phase per rotation, one wave per workgroup with
// counters before and this now: mixed spectra n = 512 2.03 -> 1.58 us, 1024 2.20 -> 1.64, 2500
// (nearly diagonal) 2.11 -> 1.77; tight cluster n = 600 4.06 -> 3.20.
template <bool GAP>
__global__ __launch_bounds__(256) void k_jacobi_spec4(JDesc d, long long log_base, MwCtl* mc,
                                                      double* xb, int G) {
  constexpr int K = 8, SW = 4;
  if (blockIdx.x % kMwStride) return;
  const int g = blockIdx.x / kMwStride;
  if (g >= G) return;
  extern __shared__ double s_diag[];
  __shared__ double s_new[K][4][kWave];  // of stage j: scores p, q, new entries p, q
  __shared__ int s_start;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = d.n, ld = d.ld;
  const int k = g * kWave + lane, kc = min(k, n - 1);
  double* A = d.A;
  auto ld_a = [&](int r, int c) -> double { return ld_ag(A + (size_t)r * ld + c); };
  auto st_a = [&](int r, int c, double v) { st_ag(A + (size_t)r * ld + c, v); };

  if (wv == 0) {
    const bool ok = mw_start(mc, G, g, 1);
    if (lane == 0) s_start = ok;
  }
  for (int l = tid; l < n; l += 256) s_diag[l] = d.diag[l];
  __syncthreads();
  if (!s_start) return;

  double dk = 0.0, bs = -1.0, bv = 0.0, bu = -1.0;
  int ba = -1, bst = 0, tk = 0;
  if (k < n) {
    dk = d.diag[k]; bs = d.bs[k]; ba = d.ba[k]; bv = d.bv[k]; bst = d.bst[k];
    bu = d.bu[k]; tk = d.ts[k];
  }
  long long rot = d.ctl->rotations, rescans = 0;
  int status = ST_OK, done = 0, kmax = K, round = 1, votes = 0;
  const double thr = d.thr;
  double wsel = 0.0;
  long long tph[6] = {0, 0, 0, 0, 0, 0}, tmark = 0;
  const bool prof = d.prof != nullptr && g == 0 && wv == 0;
  auto lap = [&](int i) {
    if (prof) {
      const long long t = (long long)wall_clock64();
      tph[i] += t - tmark;
      tmark = t;
    }
  };
  // waits until every workgroup's word has reached `want` (in its high bits) and returns this
  // lane's; -1 after a wait ran out
  const int wi = min(lane, G - 1);
  auto wait_all = [&](int* words, int want, int shift) -> int {
    for (int outer = 0; outer < kMwSpinLimit / 64 && !ld_ag_i(&mc->abort); ++outer) {
#pragma unroll 1
      for (int spins = 0; spins < 64; ++spins) {
        const int v = ld_ag_i(words + wi);
        if (!__ballot((v >> shift) < want)) {
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          return v;
        }
      }
    }
    if (lane == 0) st_ag_i(&mc->abort, 1);
    return -1;
  };
  auto uni = [](int v) -> int { return __builtin_amdgcn_readfirstlane(v); };
  // every store of this workgroup's waves is in L2, then its flag is raised
  auto arrive = [&]() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) st_word(&mc->flag[g], round);
  };

  for (;;) {
    if (prof) tmark = (long long)wall_clock64();
    // ---- publish the best candidate of every 16 lanes
    ++round;
    double* slots = xb + (size_t)(round & 1) * kMwMaxGroups * 16;
    if (wv == 0) {
      const int rc0 = k | (ba & 0x1fff) << 13 | bst << 26;
      const double s0 = bs >= 0.0 ? bs : -1.0 - lane;
      if (row_best(s0, scand_key(rc0))) {
        double* p = slots + 4 * (4 * g + (lane >> 4));
        st_ag(p, s0);
        st_ag(p + 1, bv);
        st_ag(p + 2, __longlong_as_double((long long)rc0));
      }
    }
    lap(0);
    arrive();
    if (wait_all(mc->flag, round, 0) < 0) return;
    lap(1);
    // ---- the best of this lane's share of the candidates
    SCand y = empty_scand();
    {
      SCand z[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        z[u] = empty_scand();
        if (u * 16 < G && lane + 64 * u < 4 * G) {
          const double* p = slots + 4 * (lane + 64 * u);
          z[u].s = ld_ag(p);
          z[u].a = ld_ag(p + 1);
          z[u].rc = (int)__double_as_longlong(ld_ag(p + 2));
        }
      }
      int yk = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int zk = scand_key(z[u].rc);
        if (z[u].s >= 0.0 && better(z[u].s, zk, y.s, yk)) { y = z[u]; yk = zk; }
      }
    }
    // scores rounded to 17 bits, then the lane: this order picks the candidates below, and the
    // first one where no other rounds to the same value
    int order = y.s >= 0.0 ? (key32(y.s) & ~63) | (lane ^ 63) : -1;
    int w;
    {
      const int top = uni(wave_max_i(order));
      const unsigned long long same = __ballot((order | 63) == (top | 63));
      w = top < 0 ? -1 : (top & 63) ^ 63;
      if (top >= 0 && (same & (same - 1))) w = uni(wave_argmax_lane(y.s, scand_key(y.rc)));
    }
    wsel = w >= 0 ? readlane_d(y.s, w) : 0.0;  // no pair left: every entry is 0
    if (n < 2) { done = 1; break; }
    int rc = w >= 0 ? readlane_i(y.rc, w) : 0;
    // ---- the winner must be exact
    if (w >= 0 && scand_stale(rc)) {
      const int r = scand_row(rc);
      Cand c = empty_cand();
      const double v = ld_a(r, kc);
      if (k < n && k != r) cand_top2(c, sel_score<GAP>(s_diag[r], dk, v), k, v);
      Cand e1 = empty_cand(), e2 = empty_cand();
      wave_best3(e1, 0, c, c.c, e2, 0);
      ++round;
      double* bests = xb + 2 * kMwMaxGroups * 16 + (size_t)(round & 1) * kMwMaxGroups * 4;
      if (tid == 0) put_cand(bests + 4 * g, c);
      arrive();
      if (wait_all(mc->flag, round, 0) < 0) return;
      c = lane < G ? get_cand(bests + 4 * lane) : empty_cand();
      e1 = empty_cand();
      e2 = empty_cand();
      wave_best3(e1, 0, c, c.c, e2, 0);
      if (k == r) { bs = c.s; ba = c.c; bv = c.a; bu = c.u; bst = 0; }
      ++rescans;
      lap(3);
      continue;
    }
    // ---- stop rules (checked before every rotation)
    if (wsel <= thr) { done = 1; break; }
    if (rot >= d.maxrot) { status = ST_MAXROT; done = 1; break; }
    // (a score above thr >= 0 has a nonzero entry: no stall)
    if (rot - log_base >= d.log_cap) break;  // log full: drain and resume
    const long long room = min(d.maxrot - rot, d.log_cap - (rot - log_base));
    const int klim = uni((int)min((long long)kmax, room));

    // ---- candidates on rows and columns of their own: rotation j in lane j, as its lane here
    // (my, pk: the round's rotation of this row and its other row; hs: the one that moves its
    // best entry)
    int vpq = 0, vw = w, my = -1, pk = kc, hs = K, kk = 0;
    {
      const int r1 = scand_row(y.rc), c1 = scand_stale(y.rc) ? r1 : scand_col(y.rc);
      for (;;) {
        const int x0 = scand_row(rc), x1 = scand_col(rc), p = min(x0, x1), q = max(x0, x1);
        const bool here = lane == kk;
        vpq = here ? p | q << 13 : vpq;
        vw = here ? w : vw;
        const bool piv = (k == p) | (k == q);
        my = piv ? kk : my;
        pk = piv ? p + q - k : pk;
        hs = (!bst & ((ba == p) | (ba == q))) ? kk : hs;
        ++kk;
        if (kk >= klim) break;
        const bool out = (r1 == p) | (r1 == q) | (c1 == p) | (c1 == q);
        order = out ? -1 : order;
        const int top = uni(wave_max_i(order));
        if (top < 0) break;
        w = (top & 63) ^ 63;
        rc = readlane_i(y.rc, w);
        if (scand_stale(rc)) break;
      }
    }
    // the list ends where its scores do not decrease or reach the threshold
    const double vs = __shfl(y.s, vw), va = __shfl(y.a, vw);
    {
      const double vprev = __shfl_up(vs, 1);
      const unsigned long long cut = __ballot(lane > 0 && lane < kk && !(vs < vprev && vs > thr));
      if (cut) kk = uni((int)__ffsll((long long)cut) - 1);
      if (my >= kk) { my = -1; pk = kc; }
    }
    // ---- loads of this wave's stages, then the rotation parameters in lanes
    double xv[2], yv[2], px[2] = {0.0, 0.0}, py[2] = {0.0, 0.0};
    int pj[2], qj[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = wv + SW * u, pq = readlane_i(vpq, j);
      pj[u] = pq & 0x1fff;
      qj[u] = pq >> 13;
      xv[u] = yv[u] = 0.0;
      if (j < kk) {
        xv[u] = ld_a(pj[u], kc);
        yv[u] = ld_a(qj[u], kc);
        if (__ballot(my >= 0 && my < j)) {
          px[u] = ld_a(pj[u], pk);
          py[u] = ld_a(qj[u], pk);
        }
      }
    }
    lap(2);
    const double app = s_diag[vpq & 0x1fff], aqq = s_diag[vpq >> 13];
    double vt, vc, vsn;
    rot_params<double>(app, aqq, lane < kk ? va : 1.0, vt, vc, vsn);
    const double vnp = app + vt * va, vnq = aqq - vt * va;
    // this row's own rotation, for the stages after it
    double mc_ = 1.0, ms_ = 0.0, dn = dk;
    if (__ballot(my >= 0)) {
      const int src = max(my, 0);
      const double c0 = __shfl(vc, src), s0 = __shfl(vsn, src);
      const double np0 = __shfl(vnp, src), nq0 = __shfl(vnq, src);
      const bool isp = k < pk;
      if (my >= 0) {
        mc_ = c0;
        ms_ = isp ? s0 : -s0;
        dn = isp ? np0 : nq0;
      }
    }
    // ---- new entries and scores of this wave's stages
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = wv + SW * u;
      if (j < kk) {
        const double c = readlane_d(vc, j), s = readlane_d(vsn, j);
        const double np_ = readlane_d(vnp, j), nq_ = readlane_d(vnq, j);
        const bool comp = my >= 0 && my < j;
        const double xo = comp ? mc_ * xv[u] + ms_ * px[u] : xv[u];
        const double yo = comp ? mc_ * yv[u] + ms_ * py[u] : yv[u];
        const double dc = comp ? dn : dk;
        xv[u] = c * xo + s * yo;
        yv[u] = c * yo - s * xo;
        s_new[j][0][lane] = sel_score<GAP>(dc, np_, xv[u]);
        s_new[j][1][lane] = sel_score<GAP>(dc, nq_, yv[u]);
        s_new[j][2][lane] = xv[u];
        s_new[j][3][lane] = yv[u];
      }
    }
    __syncthreads();
    lap(4);
    // ---- F = rotations proven (every wave on its own copy)
    double sp[K], sq[K];
    auto proven = [&](int j0, double& e, double& ob) -> int {  // of stages j0 .. j0 + 3
      unsigned long long bad[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        sp[j0 + u] = s_new[j0 + u][0][lane];
        sq[j0 + u] = s_new[j0 + u][1][lane];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + u;
        const double next = readlane_d(vs, j + 1);
        const bool piv = my == j;
        e = (piv | (k >= n)) ? -1.0 : fmax(e, fmax(sp[j], sq[j]));
        ob = piv ? -1.0 : (hs == j ? fmin(ob, bu) : ob);
        bad[u] = __ballot(!(fmax(e, ob) < next));
      }
      int f = kk;
#pragma unroll
      for (int u = 3; u >= 0; --u)
        if (j0 + u + 1 < kk && bad[u]) f = j0 + u + 1;
      return f;
    };
    int F;
    {
      double e = -1.0;
      double ob = (my >= 0 && !bst && ba == pk) ? bu : bs;
      F = proven(0, e, ob);
      if (F > 4) F = proven(4, e, ob);
    }
    // ---- vote: the loads of this workgroup are complete (their values are in LDS), so the
    // stores that follow the vote elsewhere cannot meet them
    if (kk > 1) {
      ++votes;
      if (tid == 0) st_word(&mc->ballot[g], votes << 4 | F);
      const int v = wait_all(mc->ballot, votes, 4);
      if (v < 0) return;
      F = uni(-wave_max_i(-(v & 15)));
    }
    // ---- commit rotations 0 .. F - 1: the stores by the waves of their stages
    const bool moved = my >= 0 && my < F;  // this row's partner rows store what precedes it
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = wv + SW * u, p = pj[u], q = qj[u];
      if (j < F && k < n) {
        if (k == p) st_a(q, p, 0.0);
        else if (k == q) st_a(p, q, 0.0);
        else if (!(moved && my > j)) {
          st_a(p, k, xv[u]);
          st_a(q, k, yv[u]);
          st_a(k, p, xv[u]);
          st_a(k, q, yv[u]);
        }
      }
    }
    if (wv == 0 && lane < F) {
      const int p = vpq & 0x1fff, q = vpq >> 13;
      s_diag[p] = vnp;
      s_diag[q] = vnq;
      if (g == 0) d.log[rot - log_base + lane] = RotEntry{p, q, vc, vsn};
    }
    RowNew rn{-1.0, -1.0, 0};
#pragma unroll
    for (int j = 0; j < K; ++j) {
      if (j < F) {
        const bool in = !(moved & (my >= j));
        row_insert(rn, in ? sp[j] : -1.0, 2 * j);
        row_insert(rn, in ? sq[j] : -1.0, 2 * j + 1);
      }
    }
    if (__ballot(rn.m1 > 0.0 && rn.m1 == rn.m2)) {
      // equal best scores in a row: the smallest column
      int col = 0x7fffffff;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if (j < F) {
          const int pq = readlane_i(vpq, j);
          const bool in = !(moved & (my >= j));
          if (in && sp[j] == rn.m1 && (pq & 0x1fff) < col) { col = pq & 0x1fff; rn.code = 2 * j; }
          if (in && sq[j] == rn.m1 && (pq >> 13) < col) { col = pq >> 13; rn.code = 2 * j + 1; }
        }
      }
    }
    {
      const int pq = __shfl(vpq, rn.code >> 1);
      const double a = s_new[rn.code >> 1][2 + (rn.code & 1)][lane];
      if (k < n) {
        if (moved) {
          dk = dn;
          tk = (int)(rot + my + 1);
        }
        const bool up = row_refresh(bs, ba, bu, bst, moved, hs < F, rn,
                                    rn.code & 1 ? pq >> 13 : pq & 0x1fff);
        bv = up ? a : bv;
      }
    }
    rot += F;
    kmax = min(K, F + 1 + (F == kk ? 1 : 0));
    lap(5);
  }

  // ---- write the state back (a later launch may resume from it)
  if (wv == 0 && k < n) {
    d.diag[k] = dk; d.bs[k] = bs; d.ba[k] = ba; d.bv[k] = bv; d.bst[k] = bst;
    d.bu[k] = bu; d.ts[k] = tk;
  }
  if (prof && lane == 0)
    for (int i = 0; i < 6; ++i) d.prof[i] += tph[i];
  if (g == 0 && tid == 0) {
    JCtl* ctl = d.ctl;
    ctl->rotations = rot;
    ctl->rescans += rescans;
    ctl->status = status;
    ctl->done = done;
    ctl->final_sel = wsel;
    ctl->final_cert = GAP ? wsel : -1.0;
    ctl->final_off = 0.0;
  }
}

// Workgroups and rows per lane for n: G = ceil(n / 64) workgroups, at most 32 (one per CU of
// an XCD) for one rotation per exchange and 64 for speculative rounds, where the scores of a
// round bound the wave; RM rows per lane (1, 2 or 4).
void mw_shape(int n, bool spec, int* G, int* RM) {
  int g = (n + kWave - 1) / kWave;
  g = std::min(g, spec ? kMwMaxGroups : kMwMaxGroups / 2);
  int rm = (n + g * kWave - 1) / (g * kWave);
  if (rm == 3) rm = 4;
  *G = g;
  *RM = rm;
}

size_t mw_bytes(int n) {
  int G, RM;
  mw_shape(n, false, &G, &RM);
  const size_t one = (size_t)2 * G * kMwWords;  // one rotation per exchange
  // (2 x 4 candidates of four words a workgroup and two rows' bests of four: both forms)
  const size_t spec = 2 * kMwMaxGroups * 16 + (size_t)2 * kMwMaxGroups * 4;
  return sizeof(MwCtl) + std::max(one, spec) * sizeof(double);
}

// The speculative loop covers every case but two, whose stop rules need more than the best
// pivot after each rotation: the off-norm stop, and greedy pivots with the certificate.
template <int RM, bool GAP>
static hipError_t launch_mw_t(const JDesc& d, long long log_base, int G, MwCtl* mc, double* xb,
                              hipStream_t s) {
  const size_t sh = (size_t)d.n * sizeof(double);
  auto fn = k_jacobi_mw<RM, GAP>;
  int threads = kWave;
  if (jacobi_speculates(d.pivot, d.stop)) {
    if constexpr (RM == 1) {
      fn = k_jacobi_spec4<GAP>;
      threads = 4 * kWave;
    } else if constexpr (RM == 2) {
      fn = k_jacobi_spec_mw<2, 4, GAP>;
    }
  }
  if (sh > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)fn,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
  }
  hipError_t e = launch_zero_words(mc, (int)(sizeof(MwCtl) / 4), s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fn, dim3(G * kMwStride), dim3(threads), sh, s, d, log_base, mc, xb, G);
  return hipGetLastError();
}

hipError_t launch_jacobi_mw(const JDesc& d, long long log_base, void* buf, hipStream_t s) {
  int G, RM;
  mw_shape(d.n, jacobi_speculates(d.pivot, d.stop), &G, &RM);
  // every row needs an owner thread
  if ((long long)G * kWave * RM < d.n || G > kMwMaxGroups) return hipErrorInvalidValue;
  MwCtl* mc = (MwCtl*)buf;
  double* xb = (double*)((char*)buf + sizeof(MwCtl));
  if (d.pivot == 1) {
    if (RM == 1) return launch_mw_t<1, true>(d, log_base, G, mc, xb, s);
    if (RM == 2) return launch_mw_t<2, true>(d, log_base, G, mc, xb, s);
    return launch_mw_t<4, true>(d, log_base, G, mc, xb, s);
  }
  if (RM == 1) return launch_mw_t<1, false>(d, log_base, G, mc, xb, s);
  if (RM == 2) return launch_mw_t<2, false>(d, log_base, G, mc, xb, s);
  return launch_mw_t<4, false>(d, log_base, G, mc, xb, s);
}

}  // namespace je
