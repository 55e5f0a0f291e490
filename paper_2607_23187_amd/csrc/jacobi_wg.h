// The FP64 pivoted Jacobi phase of one matrix in one workgroup (Algorithm 1): the loop that
// exchanges candidates after every rotation, and the speculative one (jacobi_spec.h).  Layout
// of A and the per-row caches: jacobi_kernels.hip.  Included by the single-problem and the
// batched kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "jacobi_device.h"
#include "jacobi_spec.h"
#include "kernels.h"

namespace je {

// ------------------------------------------------------------------ J1..J6: pivoted Jacobi
// Slot indices of the per-wave partial results exchanged through LDS.
enum {
  SL_SEL = 0,   // best cached selection candidate over the wave's rows (rows p, q excluded)
  SL_RP = 1,    // new row p: best (score, column) and bound of its other scores
  SL_RQ = 2,    // new row q
  SL_CERT = 3,  // best cached certificate value (greedy) over the wave's rows
  SL_CP = 4,    // new row p, certificate
  SL_CQ = 5,    // new row q, certificate
  SL_N = 6
};

template <int NW>
struct Slots {
  Cand c[2][SL_N][NW];
  double sum[2][3][NW];  // off2 of the wave's rows, of the new row p, of the new row q
};

// Cross-wave reduction of three slot groups at once: lane 16 g + w holds entry w of group
// g (g = 0, 1, 2; w < NW <= 16).  One DPP butterfly inside each 16-lane row yields the
// three group maxima; ties of the float keys are settled exactly.  Group 0 is keyed by
// row, groups 1 and 2 by column; for groups 1 and 2 u bounds every value but the winner's.
template <int NW>
__device__ __forceinline__ void reduce_groups3(const Cand* g0, const Cand* g1, const Cand* g2,
                                               Cand& r0, Cand& r1, Cand& r2) {
  const int lane = lane_id();
  const int grp = lane >> 4, w = lane & 15;
  Cand x = empty_cand();
  if (w < NW && grp < 3) x = (grp == 0 ? g0 : (grp == 1 ? g1 : g2))[w];
  const int key = (grp == 0) ? x.i : x.c;
  const int k32 = key32(x.s);
  int m = k32;
  m = max(m, dpp_i<0xB1>(m));
  m = max(m, dpp_i<0x4E>(m));
  m = max(m, dpp_i<0x141>(m));
  m = max(m, dpp_i<0x140>(m));
  const unsigned long long hit = __ballot(k32 == m && x.s >= 0.0);
  int win[3];
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    unsigned long long b = hit & (0xffffull << (16 * g));
    int wl = b ? __ffsll((long long)b) - 1 : -1;
    if (b & (b - 1)) {  // equal float keys: exact comparison
      double bs = readlane_d(x.s, wl);
      int bk = readlane_i(key, wl);
      b &= b - 1;
      while (b) {
        int l = __ffsll((long long)b) - 1;
        b &= b - 1;
        double v = readlane_d(x.s, l);
        int kv = readlane_i(key, l);
        if (v > bs || (v == bs && kv < bk)) { bs = v; bk = kv; wl = l; }
      }
    }
    win[g] = wl;
  }
  // bound of the other values in groups 1 and 2: the winner offers its u, the rest their s
  const bool mine = (grp == 1 && lane == win[1]) || (grp == 2 && lane == win[2]);
  int mu = key32(mine ? x.u : x.s);
  mu = max(mu, dpp_i<0xB1>(mu));
  mu = max(mu, dpp_i<0x4E>(mu));
  mu = max(mu, dpp_i<0x141>(mu));
  mu = max(mu, dpp_i<0x140>(mu));
  const int mu1 = readlane_i(mu, 16), mu2 = readlane_i(mu, 32);
  r0 = read_cand(x, win[0], false);
  r1 = read_cand(x, win[1], false);
  r2 = read_cand(x, win[2], false);
  r1.u = key_ub(mu1);
  r2.u = key_ub(mu2);
}

// Cross-wave argmax of slot k over the NW waves: every lane scans the same NW entries
// (broadcast LDS reads), keeping the first maximum in (score desc, key asc) order; u is
// the bound of all values but the winner's.
template <int NW>
__device__ __forceinline__ Cand reduce_slot(const Slots<NW>& S, int b, int k, bool by_col) {
  Cand best = S.c[b][k][0];
  int bw = 0;
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    const Cand x = S.c[b][k][w];
    const int kx = by_col ? x.c : x.i, kb = by_col ? best.c : best.i;
    if (better(x.s, kx, best.s, kb)) { best = x; bw = w; }
  }
  double u = best.u;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w != bw) u = fmax(u, S.c[b][k][w].s);
  best.u = u;
  return best;
}

template <int NW>
__device__ __forceinline__ double reduce_sum_slot(const Slots<NW>& S, int b, int k) {
  double v = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) v += S.sum[b][k][w];  // fixed order: wave 0, 1, ...
  return v;
}

// NT threads (NW waves), RM rows per thread (row k = tid + i * NT).  LDSA: A lives in
// LDS.  MIR: columns p and q are stored as well (mirrored update; rows are then always
// current and every load is a contiguous row segment); otherwise rows only, with the
// per-row write timestamps choosing the current copy of each entry.
template <int NT, int RM, bool GAP, bool LDSA, bool MIR>
__device__ __forceinline__ void jacobi_body(const JDesc d, long long log_base) {
  constexpr int NW = NT / kWave;
  extern __shared__ double smem[];
  __shared__ Slots<NW> S;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
  const int n = d.n;
  const bool use_cert = !GAP && d.stop == STOP_CERT;
  const bool use_off = d.stop == STOP_OFF;

  double* s_diag = smem;
  int* s_ts = reinterpret_cast<int*>(s_diag + n);
  double* s_A = s_diag + n + (n + 1) / 2;  // after the int array, 8-byte aligned
  const int ldl = n | 1;
  const int ld = d.ld;
  double* gA = d.A;

  auto ld_a = [&](int r, int c) -> double {
    if constexpr (LDSA) return s_A[r * ldl + c];
    else return gA[(size_t)r * ld + c];
  };
  auto st_a = [&](int r, int c, double v) {
    if constexpr (LDSA) s_A[r * ldl + c] = v;
    else gA[(size_t)r * ld + c] = v;
  };
  auto sync = [&]() {
    if constexpr (NW > 1) __syncthreads();
  };

  // ---- per-thread rows k = tid + i * NT
  double dk[RM], bs[RM], bv[RM], bu[RM], cb[RM], cu[RM], of2[RM];
  int ba[RM], bst[RM], ca[RM], cst[RM], tk[RM];
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    int k = tid + i * NT;
    if (k < n) {
      dk[i] = d.diag[k]; bs[i] = d.bs[k]; ba[i] = d.ba[k]; bv[i] = d.bv[k]; bst[i] = d.bst[k];
      bu[i] = d.bu[k]; of2[i] = d.off2[k]; tk[i] = d.ts[k];
      if (use_cert) { cb[i] = d.cb[k]; ca[i] = d.ca[k]; cst[i] = d.cst[k]; cu[i] = d.cu[k]; }
      else { cb[i] = -1.0; ca[i] = -1; cst[i] = 0; cu[i] = -1.0; }
      s_diag[k] = dk[i];
      s_ts[k] = tk[i];
    } else {
      dk[i] = 0.0; bs[i] = -1.0; ba[i] = -1; bv[i] = 0.0; bst[i] = 0; bu[i] = -1.0; of2[i] = 0.0;
      tk[i] = 0; cb[i] = -1.0; ca[i] = -1; cst[i] = 0; cu[i] = -1.0;
    }
  }
  if constexpr (LDSA) {
    for (int idx = tid; idx < n * n; idx += NT) {
      int r = idx / n, c = idx - r * n;
      s_A[r * ldl + c] = gA[(size_t)r * ld + c];
    }
  }
  __syncthreads();

  long long rot = d.ctl->rotations;
  long long rescans = 0;
  int status = ST_OK, done = 0;
  const double thr = d.thr;
  // last rotation (its diagonal entries and timestamps reach LDS one iteration later)
  int lp = -1, lq = -1, lrot = 0;
  double lapp = 0.0, laqq = 0.0;
  bool pend = false;
  // per-thread top two of the new rows p and q (filled by a rotation)
  Cand rp = empty_cand(), rq = rp, cp = rp, cq = rp;
  double op = 0.0, oq = 0.0;
  Cand W = empty_cand(), C = empty_cand();
  double off_tot = 0.0;
  int it = 0;

  auto diag_of = [&](int x) -> double { return x == lp ? lapp : (x == lq ? laqq : s_diag[x]); };
  auto ts_of = [&](int x) -> int { return (x == lp || x == lq) ? lrot : s_ts[x]; };
  // current value of entry (r, l), l owned by this thread with timestamp tl
  auto entry = [&](int r, int l, int tl, int tr) -> double {
    if constexpr (MIR) return ld_a(r, l);
    else return (tl > tr) ? ld_a(l, r) : ld_a(r, l);
  };
  // optional phase timers: wave reductions, barrier, cross-wave, rescans, rotation
  const bool prof = d.prof != nullptr;
  long long tw = 0, tb = 0, tx = 0, tr = 0, tp = 0, tu = 0, tmark = 0;
  auto tick = [&]() -> long long { return prof ? (long long)wall_clock64() : 0; };
  const long long clk0 = prof ? (long long)clock64() : 0, wall0 = tick();

  // Full rescan of row r's selection (which == 0) or certificate (which == 1) cache:
  // exact best and the bound of the other scores.
  auto rescan = [&](int r, int which) {
    const int b = it & 1;
    const double arr = diag_of(r);
    const int trr = MIR ? 0 : ts_of(r);
    double vals[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int l = tid + i * NT;
      vals[i] = (l < n && l != r) ? entry(r, l, tk[i], trr) : 0.0;
    }
    Cand x = empty_cand();
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int l = tid + i * NT;
      if (l >= n || l == r) continue;
      double v = vals[i];
      double sc = which == 0 ? sel_score<GAP>(arr, dk[i], v) : gap_score(arr, dk[i], v);
      cand_top2(x, sc, l, v);
    }
    Cand e1 = empty_cand(), e2 = empty_cand();
    wave_best3(e1, 0, x, x.c, e2, 0);
    if (NW > 1) {
      if (lane == 0) S.c[b][SL_RP][wid] = x;
      __syncthreads();
      x = reduce_slot(S, b, SL_RP, true);
    }
    ++it;
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      if (tid + i * NT == r) {
        if (which == 0) { bs[i] = x.s; ba[i] = x.c; bv[i] = x.a; bu[i] = x.u; bst[i] = 0; }
        else { cb[i] = x.s; ca[i] = x.c; cu[i] = x.u; cst[i] = 0; }
      }
    }
    ++rescans;
  };

  for (;;) {
    const int b = it & 1;
    tmark = tick();
    // ---- per-thread candidates over own rows
    Cand x1 = empty_cand(), x4 = empty_cand();
    double o7 = 0.0;
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int k = tid + i * NT;
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
    if (prof) { long long t = tick(); tw += t - tmark; tmark = t; }
    if constexpr (NW > 1) {
      if (lane == 0) {
        S.c[b][SL_SEL][wid] = w1; S.c[b][SL_RP][wid] = w2; S.c[b][SL_RQ][wid] = w3;
        if (use_cert) { S.c[b][SL_CERT][wid] = w4; S.c[b][SL_CP][wid] = w5; S.c[b][SL_CQ][wid] = w6; }
        if (use_off) { S.sum[b][0][wid] = s7; S.sum[b][1][wid] = s8; S.sum[b][2][wid] = s9; }
      }
      __syncthreads();
      if (prof) { long long t = tick(); tb += t - tmark; tmark = t; }
      reduce_groups3<NW>(S.c[b][SL_SEL], S.c[b][SL_RP], S.c[b][SL_RQ], w1, w2, w3);
      if (use_cert)
        reduce_groups3<NW>(S.c[b][SL_CERT], S.c[b][SL_CP], S.c[b][SL_CQ], w4, w5, w6);
      if (use_off) {
        s7 = reduce_sum_slot(S, b, 0);
        s8 = reduce_sum_slot(S, b, 1);
        s9 = reduce_sum_slot(S, b, 2);
      }
    }
    ++it;
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
        int k = tid + i * NT;
        if (k == lp) {
          bs[i] = w2.s; ba[i] = w2.c; bv[i] = w2.a; bu[i] = w2.u; bst[i] = 0; of2[i] = s8;
          if (use_cert) { cb[i] = w5.s; ca[i] = w5.c; cu[i] = w5.u; cst[i] = 0; }
        } else if (k == lq) {
          bs[i] = w3.s; ba[i] = w3.c; bv[i] = w3.a; bu[i] = w3.u; bst[i] = 0; of2[i] = s9;
          if (use_cert) { cb[i] = w6.s; ca[i] = w6.c; cu[i] = w6.u; cst[i] = 0; }
        }
      }
      if (tid == 0) {
        s_diag[lp] = lapp; s_diag[lq] = laqq;
        s_ts[lp] = lrot; s_ts[lq] = lrot;
      }
      pend = false;
      rp = empty_cand(); rq = rp; cp = rp; cq = rp;
      op = 0.0; oq = 0.0;
    }
    if (prof) { long long t = tick(); tx += t - tmark; tmark = t; }
    if (n < 2) { done = 1; break; }
    // ---- the winner must be exact
    if (W.f) {
      rescan(W.i, 0);
      if (prof) { long long t = tick(); tr += t - tmark; }
      continue;
    }
    // ---- stop rules (checked before every rotation)
    if (d.stop == STOP_CERT) {
      if (GAP) {
        if (W.s <= thr) { done = 1; break; }
      } else {
        if (C.s <= thr) { done = 1; break; }
        if (C.f) {
          rescan(C.i, 1);
          if (prof) { long long t = tick(); tr += t - tmark; }
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
    const int tsp = MIR ? 0 : ts_of(p), tsq = MIR ? 0 : ts_of(q);
    double xv[RM], yv[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int k = tid + i * NT;
      xv[i] = 0.0; yv[i] = 0.0;
      if (k >= n || k == p || k == q) continue;
      xv[i] = entry(p, k, tk[i], tsp);
      yv[i] = entry(q, k, tk[i], tsq);
    }
    const double apq = W.a;
    const double app = diag_of(p), aqq = diag_of(q);
    double t, c, s;
    rot_params<double>(app, aqq, apq, t, c, s);
    const double napp = app + t * apq;
    const double naqq = aqq - t * apq;
    const int nts = (int)(rot + 1);
    if (prof) { long long tt = tick(); tp += tt - tmark; tmark = tt; }
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      int k = tid + i * NT;
      if (k >= n) continue;
      if (k == p) {
        st_a(q, p, 0.0);
        if (MIR) st_a(p, q, 0.0);
        dk[i] = napp; tk[i] = nts;
        cand_top2(rq, 0.0, p, 0.0);
        if (use_cert) cand_top2(cq, 0.0, p, 0.0);
        continue;
      }
      if (k == q) {
        if (!MIR) st_a(p, q, 0.0);
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
      if (MIR) { st_a(k, p, xn); st_a(k, q, yn); }
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
    if (tid == 0) d.log[rot - log_base] = RotEntry{p, q, c, s};
    if (prof) { long long tt = tick(); tu += tt - tmark; }
    lp = p; lq = q; lapp = napp; laqq = naqq; lrot = nts;
    pend = true;
    ++rot;
  }

  // ---- write the state back (a later launch may resume from it)
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    int k = tid + i * NT;
    if (k < n) {
      d.diag[k] = dk[i]; d.bs[k] = bs[i]; d.ba[k] = ba[i]; d.bv[k] = bv[i]; d.bst[k] = bst[i];
      d.bu[k] = bu[i]; d.off2[k] = of2[i]; d.ts[k] = tk[i];
      if (use_cert) { d.cb[k] = cb[i]; d.ca[k] = ca[i]; d.cst[k] = cst[i]; d.cu[k] = cu[i]; }
    }
  }
  if constexpr (LDSA) {
    if (!done) {
      __syncthreads();
      for (int idx = tid; idx < n * n; idx += NT) {
        int r = idx / n, c = idx - r * n;
        gA[(size_t)r * ld + c] = s_A[r * ldl + c];
      }
    }
  }
  if (prof && tid == 0) {
    d.prof[0] += tw; d.prof[1] += tb; d.prof[2] += tx; d.prof[3] += tr; d.prof[4] += tp;
    d.prof[5] += tu;
    d.prof[6] += (long long)clock64() - clk0;
    d.prof[7] += tick() - wall0;
  }
  if (tid == 0) {
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
// The exchange of the speculative loop (jacobi_spec.h) inside one workgroup: candidates,
// votes and the diagonal through LDS, two barriers a round.  One wave (NW = 1) needs none.
template <int NW>
struct SpecShared {
  double s[NW * 4], a[NW * 4];
  int rc[NW * 4];
  int vote[NW];
  Cand best[NW];
};

template <int NW, bool LDSA, bool MIR>
struct WgExchange {
  static constexpr bool kExchange = NW > 1;
  SpecShared<NW>& S;
  double* A;         // LDS or device memory
  double* s_diag;
  int* s_ts;
  int T, GT, ld_, lane, wid;

  __device__ __forceinline__ bool first_wave() const { return wid == 0; }
  __device__ __forceinline__ bool ok() const { return true; }
  // one wave: its own LDS accesses complete in order, only the compiler has to keep them so
  __device__ __forceinline__ void fence() const { __atomic_signal_fence(__ATOMIC_SEQ_CST); }
  __device__ __forceinline__ void publish(bool win, const SCand& x) {
    if (win) {
      const int i = 4 * wid + (lane >> 4);
      S.s[i] = x.s;
      S.a[i] = x.a;
      S.rc[i] = x.rc;
    }
  }
  __device__ __forceinline__ SCand gather(const SCand& x) {
    SCand y = x;
    if constexpr (NW == 1) {
      fence();
    } else {
      __syncthreads();
      y = empty_scand();
      if (lane < 4 * NW) y = SCand{S.s[lane], S.a[lane], S.rc[lane]};
    }
    return y;
  }
  __device__ __forceinline__ int vote(int F, int kk) {
    if constexpr (NW == 1) {
      fence();
      return F;
    } else {
      // the loads of this round are complete: the stores after the vote go to the same rows
      if constexpr (!LDSA) __builtin_amdgcn_s_waitcnt(0);
      if (lane == 0) S.vote[wid] = F;
      __syncthreads();
      return -wave_max_i(lane < NW ? -S.vote[lane] : -kk);
    }
  }
  __device__ __forceinline__ Cand best(const Cand& x) {
    if constexpr (NW == 1) return x;
    if (lane == 0) S.best[wid] = x;
    __syncthreads();
    Cand y = lane < NW ? S.best[lane] : empty_cand();
    Cand e1 = empty_cand(), e2 = empty_cand();
    wave_best3(e1, 0, y, y.c, e2, 0);
    return y;
  }
  __device__ __forceinline__ double ld(int r, int k, int tk) const {
    if constexpr (MIR) return A[(size_t)r * ld_ + k];
    else return tk > s_ts[r] ? A[(size_t)k * ld_ + r] : A[(size_t)r * ld_ + k];
  }
  __device__ __forceinline__ double ld2(int r, int l) const { return ld(r, l, MIR ? 0 : s_ts[l]); }
  __device__ __forceinline__ void st(int r, int k, double v) { A[(size_t)r * ld_ + k] = v; }
  __device__ __forceinline__ void stm(int k, int r, double v) {
    if constexpr (MIR) A[(size_t)k * ld_ + r] = v;
  }
  __device__ __forceinline__ double diag(int k) const { return s_diag[k]; }
  __device__ __forceinline__ void set_diag(int p, int q, double dp, double dq, int ts) {
    if (wid) return;
    s_diag[p] = dp;
    s_diag[q] = dq;
    if constexpr (!MIR) s_ts[p] = s_ts[q] = ts;
  }
};

template <int NT, int RM, int K, bool GAP, bool LDSA, bool MIR>
__device__ __forceinline__ void jacobi_spec_body(const JDesc d, long long log_base) {
  constexpr int NW = NT / kWave;
  extern __shared__ double smem[];
  __shared__ SpecShared<NW> S;
  const int tid = threadIdx.x, n = d.n;
  double* s_diag = smem;
  int* s_ts = reinterpret_cast<int*>(s_diag + n);
  double* s_A = s_diag + n + (n + 1) / 2;
  const int ldl = n | 1;
  for (int k = tid; k < n; k += NT) {
    s_diag[k] = d.diag[k];
    s_ts[k] = d.ts[k];
  }
  if constexpr (LDSA) {
    for (int idx = tid; idx < n * n; idx += NT) {
      const int r = idx / n, c = idx - r * n;
      s_A[r * ldl + c] = d.A[(size_t)r * d.ld + c];
    }
  }
  __syncthreads();
  WgExchange<NW, LDSA, MIR> ex{S, LDSA ? s_A : d.A, s_diag, s_ts, tid, NT, LDSA ? ldl : d.ld,
                               tid & (kWave - 1), tid / kWave};
  const bool done = spec_loop<RM, K, GAP>(d, log_base, ex);
  if constexpr (LDSA) {
    if (!done) {
      __syncthreads();
      for (int idx = tid; idx < n * n; idx += NT) {
        const int r = idx / n, c = idx - r * n;
        d.A[(size_t)r * d.ld + c] = s_A[r * ldl + c];
      }
    }
  }
}

// Rotations tried per round (0: one at a time): what the registers of a lane hold for its
// rows, with fewer in a batch, where several workgroups share a CU.
template <int RM, bool QUEUE>
constexpr int spec_depth() {
  return RM == 1 ? (QUEUE ? 4 : 8) : (RM == 2 ? 4 : (RM == 4 ? 2 : 0));
}

// SPEC: the speculative loop (jacobi_speculates), else one rotation per exchange.  With eight
// rows per lane only the latter fits the registers.
template <int NT, int RM, bool GAP, bool LDSA, bool MIR, bool QUEUE, bool SPEC>
__device__ __forceinline__ void jacobi_run(const JDesc d, long long log_base) {
  constexpr int K = spec_depth<RM, QUEUE>();
  if constexpr (SPEC && K > 0) jacobi_spec_body<NT, RM, K, GAP, LDSA, MIR>(d, log_base);
  else jacobi_body<NT, RM, GAP, LDSA, MIR>(d, log_base);
}

// LDS budget of the kernel's dynamic part (diagonal, timestamps, and A if LDS-resident).
inline size_t jacobi_lds_bytes(int n, bool ldsa) {
  size_t b = (size_t)n * 8 + (size_t)((n + 1) / 2) * 8;
  if (ldsa) b += (size_t)n * (size_t)(n | 1) * 8;
  return b;
}

}  // namespace je
