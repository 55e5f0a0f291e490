// Speculative form of the FP64 pivoted Jacobi loop (Algorithm 1): several rotations of the
// sequence per exchange of candidates.  Included by the kernel files only.
//
// What bounds the loop is a chain of latencies per rotation (candidate reductions, the
// exchange between waves, row loads, the FP64 square roots and divisions), not bandwidth or
// issue.  Consecutive pivots mostly touch different rows and columns: on preconditioned
// matrices the next pivots are, for three to five rotations on average, the best remaining
// candidates that were known before the first of them.  So a round
//   1. takes the best candidate, which is the exact pivot, and behind it up to K - 1 of the
//      best published candidates on rows and columns of their own, in descending order;
//   2. loads the rows of all of them, evaluates their rotation parameters in K lanes at once
//      and, in the order of the sequence, the new entries and scores, in registers;
//   3. finds the first stage j after which candidate j + 1 is not provably the next pivot:
//      some score or bound of a score is not below it;
//   4. stores the entries and refreshes the caches of the rotations before that stage.
// The rotations performed, and every value stored, are those of one rotation at a time.
//
// Row caches (Sec. 3.2) cover each pair (k, l) in row k, in row l, or in both: a rotation
// (p, q) empties rows p and q, whose new entries every other row k has just taken into its
// own cache.  So no argmax over the new rows is needed.  A full rescan of a stale row makes
// it cover all its pairs again.  Ties go to the lexicographically smallest pair; a stale row
// (an upper bound) goes before equal exact scores, so it is rescanned first.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "jacobi_device.h"
#include "kernels.h"

namespace je {

// A candidate as the rounds exchange it: score (negative: none), entry, and the packed row,
// column (< 2^13 each) and stale flag.
struct SCand {
  double s, a;
  int rc;
};

__device__ __forceinline__ SCand empty_scand() { return SCand{-1.0, 0.0, 0}; }
__device__ __forceinline__ int scand_row(int rc) { return rc & 0x1fff; }
__device__ __forceinline__ int scand_col(int rc) { return (rc >> 13) & 0x1fff; }
__device__ __forceinline__ int scand_stale(int rc) { return rc >> 26; }
// order among equal scores: stale rows first, then the pair (smaller index, larger index)
__device__ __forceinline__ int scand_key(int rc) {
  const int r = scand_row(rc), c = scand_col(rc);
  return scand_stale(rc) ? -1 : (min(r, c) << 13 | max(r, c));
}

// True in one lane of every 16: the one with the largest score, the smallest key among equal
// scores, the lowest lane among equal pairs.
__device__ __forceinline__ bool row_best(double s, int key) {
  double m = s;
  m = fmax(m, dpp_d<0xB1>(m));
  m = fmax(m, dpp_d<0x4E>(m));
  m = fmax(m, dpp_d<0x141>(m));
  m = fmax(m, dpp_d<0x140>(m));
  bool win = s == m;
  if (__popcll(__ballot(win)) > 4) {
    int k = win ? key : 0x7fffffff;
    k = min(k, dpp_i<0xB1>(k));
    k = min(k, dpp_i<0x4E>(k));
    k = min(k, dpp_i<0x141>(k));
    k = min(k, dpp_i<0x140>(k));
    const unsigned long long b = __ballot(win && key == k);
    const int lane = lane_id();
    win = (b >> lane & 1) && !(b >> (lane & 48) & ((1ull << (lane & 15)) - 1));
  }
  return win;
}

// A row's cache after a round.  The round's new entries of the row are inserted one by one into a
// running best and second best, and the cache is refreshed once from those: the outcome is a
// fresh cache (its exact best, a bound of the others) or a stale one (a bound of all), as one
// refresh per rotation would leave, in a third of the instructions.
struct RowNew {
  double m1, m2;  // best and second best new score
  int code;       // of the best: 2 * rotation + (1 for the entry in column q)
};

__device__ __forceinline__ void row_insert(RowNew& x, double v, int code) {
  x.code = v > x.m1 ? code : x.code;
  x.m2 = fmax(x.m2, fmin(x.m1, v));
  x.m1 = fmax(x.m1, v);
}

// empty: the row was rotated in the round (x holds what followed); hit: its best entry's column
// was.  True when the best new entry (column col) is the row's best now.
__device__ __forceinline__ bool row_refresh(double& bs, int& ba, double& bu, int& bst, bool empty,
                                            bool hit, const RowNew& x, int col) {
  const double bound = empty ? -1.0 : (bst ? bs : bu);
  const bool nobest = empty | (bst != 0) | hit;
  const bool up = nobest ? x.m1 > bound : better(x.m1, col, bs, ba);
  const double under = up ? fmax(x.m2, nobest ? -1.0 : bs) : (nobest ? -1.0 : x.m1);
  bs = up ? x.m1 : (nobest ? bound : bs);
  bu = fmax(bound, under);
  ba = up ? col : (empty ? -1 : ba);
  bst = (nobest & !up & (bound >= 0.0)) ? 1 : 0;
  return up;
}

// The loop over one matrix.  Ex gives the exchange and the storage of A:
//   T, GT        this thread owns rows k = T + i GT, i < RM (k < n)
//   kExchange    false: one wave, which selects among its lanes' own candidates
//   publish(win, x), gather(x): the candidates of the lanes with `win` (one in 16) out; then,
//                after a barrier over all waves, the best of lane's share of them in
//   vote(F, kk)  minimum of F <= kk over all waves (a barrier over them)
//   best(x)      exact best of the waves' row-scan candidates with the bound of the rest
//   ld(r, k, tk), ld2(r, l), st(r, k, v), stm(k, r, v): entry (r, k) for an own row k, for any
//                column l; row store, mirrored store
//   diag(k), set_diag(p, q, dp, dq, ts): diagonal of A (ts: the rotation's number, for storage
//                that chooses the newer copy of an entry by it)
//   ok()         false after a wait ran out
// All of them are called in uniform control flow of the wave.
template <int RM, int K, bool GAP, class Ex>
__device__ __forceinline__ bool spec_loop(const JDesc& d, long long log_base, Ex& ex) {
  const int lane = lane_id();
  const int n = d.n;
  double dk[RM], bs[RM], bv[RM], bu[RM];
  int ba[RM], bst[RM], tk[RM];
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    const int k = ex.T + i * ex.GT;
    dk[i] = 0.0; bs[i] = -1.0; bv[i] = 0.0; bu[i] = -1.0; ba[i] = -1; bst[i] = 0; tk[i] = 0;
    if (k < n) {
      dk[i] = d.diag[k]; bs[i] = d.bs[k]; ba[i] = d.ba[k]; bv[i] = d.bv[k]; bst[i] = d.bst[k];
      bu[i] = d.bu[k]; tk[i] = d.ts[k];
    }
  }
  long long rot = d.ctl->rotations;
  long long rescans = 0;
  int status = ST_OK, done = 0;
  const double thr = d.thr;
  double wsel = 0.0;
  // rotations tried per round: one more than the last round performed, two if it performed
  // all it tried (a stage that is not proven costs its scores; on a spectrum whose next pivot
  // mostly lies in the rows just rotated three tries in four fail)
  int kmax = K;
  long long tph[6] = {0, 0, 0, 0, 0, 0}, tmark = 0;
  const bool prof = d.prof != nullptr && ex.first_wave();
  auto lap = [&](int k) {
    if (prof) {
      const long long t = (long long)wall_clock64();
      tph[k] += t - tmark;
      tmark = t;
    }
  };

  for (;;) {
    if (prof) tmark = (long long)wall_clock64();
    // ---- best candidate of every 16 lanes (a lane without one holds a value of its own)
    SCand x = SCand{-1.0 - lane, 0.0, 0};
    {
      int xk = 0;
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        const int rc = (ex.T + i * ex.GT) | (ba[i] & 0x1fff) << 13 | bst[i] << 26;
        const int key = scand_key(rc);
        if (bs[i] >= 0.0 && better(bs[i], key, x.s, xk)) {
          x = SCand{bs[i], bv[i], rc};
          xk = key;
        }
      }
      if constexpr (Ex::kExchange) ex.publish(row_best(x.s, xk), x);
    }
    lap(0);
    // ---- exchange
    SCand y = ex.gather(x);
    if (!ex.ok()) return false;  // a wait ran out: the host reports it, the state is not resumable
    lap(1);
    int ykey = scand_key(y.rc);
    int w = wave_argmax_lane(y.s, ykey);
    wsel = w >= 0 ? readlane_d(y.s, w) : 0.0;  // no pair left: every entry is 0
    if (n < 2) { done = 1; break; }
    int rc = w >= 0 ? readlane_i(y.rc, w) : 0;
    const double a0 = w >= 0 ? readlane_d(y.a, w) : 0.0;
    // ---- the winner must be exact
    if (w >= 0 && scand_stale(rc)) {
      const int r = scand_row(rc);
      const double arr = ex.diag(r);
      double vals[RM];
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        const int l = ex.T + i * ex.GT;
        vals[i] = (l < n && l != r) ? ex.ld(r, l, tk[i]) : 0.0;
      }
      Cand c = empty_cand();
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        const int l = ex.T + i * ex.GT;
        if (l < n && l != r) cand_top2(c, sel_score<GAP>(arr, dk[i], vals[i]), l, vals[i]);
      }
      Cand e1 = empty_cand(), e2 = empty_cand();
      wave_best3(e1, 0, c, c.c, e2, 0);
      c = ex.best(c);
      if (!ex.ok()) return false;
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        if (ex.T + i * ex.GT == r) {
          bs[i] = c.s; ba[i] = c.c; bv[i] = c.a; bu[i] = c.u; bst[i] = 0;
        }
      }
      ++rescans;
      lap(3);
      continue;
    }
    // ---- stop rules (checked before every rotation)
    if (wsel <= thr) { done = 1; break; }
    if (rot >= d.maxrot) { status = ST_MAXROT; done = 1; break; }
    if (a0 == 0.0) { status = ST_STALL; done = 1; break; }
    if (rot - log_base >= d.log_cap) break;  // log full: drain and resume
    const long long room = min(d.maxrot - rot, d.log_cap - (rot - log_base));
    const int klim = (int)min((long long)kmax, room);

    // ---- candidates on rows and columns of their own, in descending order; the loads of
    // each one's rows are issued before the next is selected
    double xv[K][RM], yv[K][RM], px[K][RM], py[K][RM];
    // the round's rotation of this row and its other row; the one that moves its best entry
    int my[RM], pk[RM], hs[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) { my[i] = -1; pk[i] = min(ex.T + i * ex.GT, n - 1); hs[i] = K; }
    // rotation j in lane j: packed (p, q), score, entry
    int vpq = 0;
    double vs = 0.0, va = 0.0;
    int kk = 0;
    double sj = wsel, aj = a0, sprev = 0.0;
    // the candidates behind the first are picked by their rounded scores (17 bits, then the
    // lane); the list ends where that order is not the exact one, which the check of the stage
    // before then sees, as it sees any candidate left out
    int order = y.s >= 0.0 ? (key32(y.s) & ~63) | (lane ^ 63) : -1;
#pragma unroll
    for (int j = 0; j < K; ++j) {
#pragma unroll
      for (int i = 0; i < RM; ++i) { xv[j][i] = yv[j][i] = px[j][i] = py[j][i] = 0.0; }
      if (j == kk && j < klim) {
        if (j > 0) {
          const int m = wave_max_i(order);
          w = m < 0 ? -1 : (m & 63) ^ 63;
          if (w >= 0) {
            rc = readlane_i(y.rc, w);
            sj = readlane_d(y.s, w);
            aj = readlane_d(y.a, w);
          }
        }
        if (j == 0 ||
            (w >= 0 && !scand_stale(rc) && sj < sprev && sj > thr && aj != 0.0)) {
          const int p = min(scand_row(rc), scand_col(rc)), q = max(scand_row(rc), scand_col(rc));
          if (lane == j) { vpq = p | q << 13; vs = sj; va = aj; }
          kk = j + 1;
          sprev = sj;
#pragma unroll
          for (int i = 0; i < RM; ++i) {
            // straight-line: a pivot's own lane and lanes past n load entries they do not use
            const int k = ex.T + i * ex.GT;
            const bool piv = k == p || k == q;
            xv[j][i] = ex.ld(p, min(k, n - 1), tk[i]);
            yv[j][i] = ex.ld(q, min(k, n - 1), tk[i]);
            if (j > 0 && __ballot(my[i] >= 0)) {
              px[j][i] = ex.ld2(p, pk[i]);
              py[j][i] = ex.ld2(q, pk[i]);
            }
            my[i] = piv ? j : my[i];
            pk[i] = piv ? p + q - k : pk[i];
            hs[i] = (!bst[i] & ((ba[i] == p) | (ba[i] == q))) ? j : hs[i];
          }
          // candidates sharing a row or column with this one are out
          const int r1 = scand_row(y.rc), c1 = scand_col(y.rc);
          if (r1 == p || r1 == q || (!scand_stale(y.rc) && (c1 == p || c1 == q))) order = -1;
        }
      }
    }
    lap(2);
    // ---- rotation parameters, rotation j in lane j
    const double app = ex.diag(vpq & 0x1fff), aqq = ex.diag(vpq >> 13);
    double vt, vc, vsn;
    rot_params<double>(app, aqq, lane < kk ? va : 1.0, vt, vc, vsn);
    const double vnp = app + vt * va, vnq = aqq - vt * va;

    // ---- new entries and scores in the order of the sequence; F = rotations proven
    double sp[K][RM], sq[K][RM];
    double dc[RM], e[RM], ob[RM], mc[RM], ms[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      dc[i] = dk[i];
      e[i] = -1.0;
      // a pivot's own pair is not above itself: the bound of the row's others counts
      ob[i] = (my[i] >= 0 && !bst[i] && ba[i] == pk[i]) ? bu[i] : bs[i];
      mc[i] = 1.0;
      ms[i] = 0.0;
    }
    int F = kk;
    // stages in groups without a branch between them, so that their square roots and
    // divisions overlap
    constexpr int kGroup = 2;
#pragma unroll
    for (int j0 = 0; j0 < K; j0 += kGroup) {
      if (j0 >= F) break;
      unsigned long long bad[kGroup];
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        const int j = j0 + u;
        const double c = readlane_d(vc, j), s = readlane_d(vsn, j);
        const double np_ = readlane_d(vnp, j), nq_ = readlane_d(vnq, j);
        const double next = readlane_d(vs, j + 1);
        bool over = false;
#pragma unroll
        for (int i = 0; i < RM; ++i) {
          const int k = ex.T + i * ex.GT;
          const bool piv = my[i] == j, isp = k < pk[i];
          double xo = xv[j][i], yo = yv[j][i];
          if (j > 0) {
            // the entries as an earlier rotation of this row left them
            const bool comp = my[i] >= 0 && my[i] < j;
            const double xc = mc[i] * xo + ms[i] * px[j][i];
            const double yc = mc[i] * yo + ms[i] * py[j][i];
            xo = comp ? xc : xo;
            yo = comp ? yc : yo;
          }
          const double xn = c * xo + s * yo;
          const double yn = c * yo - s * xo;
          xv[j][i] = xn;
          yv[j][i] = yn;
          sp[j][i] = sel_score<GAP>(dc[i], np_, xn);
          sq[j][i] = sel_score<GAP>(dc[i], nq_, yn);
          const double ej = fmax(e[i], fmax(sp[j][i], sq[j][i]));
          e[i] = (piv || k >= n) ? -1.0 : ej;
          ob[i] = piv ? -1.0 : (hs[i] == j ? fmin(ob[i], bu[i]) : ob[i]);
          mc[i] = piv ? c : mc[i];
          ms[i] = piv ? (isp ? s : -s) : ms[i];
          dc[i] = piv ? (isp ? np_ : nq_) : dc[i];
          over |= !(fmax(e[i], ob[i]) < next);
        }
        bad[u] = __ballot(over);
      }
#pragma unroll
      for (int u = kGroup - 1; u >= 0; --u)
        if (j0 + u + 1 < kk && bad[u]) F = j0 + u + 1;
    }
    lap(4);
    F = ex.vote(F, kk);
    if (!ex.ok()) return false;

    // ---- commit rotations 0 .. F - 1
    RowNew rn[RM];
    double av[RM];  // the best new entry
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      rn[i] = RowNew{-1.0, -1.0, 0};
      av[i] = 0.0;
    }
    bool tie = false;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      if (j < F) {
        const int pq = readlane_i(vpq, j);
        const int p = pq & 0x1fff, q = pq >> 13;
#pragma unroll
        for (int i = 0; i < RM; ++i) {
          const int k = ex.T + i * ex.GT;
          if (k < n) {
            // (a row rotated later in the round: its partner rows store the final entries)
            const bool later = my[i] > j && my[i] < F;
            const double xn = xv[j][i], yn = yv[j][i];
            if (my[i] == j) {
              ex.st(k == p ? q : p, k, 0.0);
            } else if (!later) {
              ex.st(p, k, xn);
              ex.st(q, k, yn);
              ex.stm(k, p, xn);
              ex.stm(k, q, yn);
            }
            const bool in = my[i] != j && !later;
            const double a = in ? sp[j][i] : -1.0, b = in ? sq[j][i] : -1.0;
            av[i] = a > rn[i].m1 ? xn : av[i];
            row_insert(rn[i], a, 2 * j);
            av[i] = b > rn[i].m1 ? yn : av[i];
            row_insert(rn[i], b, 2 * j + 1);
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < RM; ++i) tie |= rn[i].m1 > 0.0 && rn[i].m1 == rn[i].m2;
    if (__ballot(tie)) {
      // equal best scores in a row: the smallest column
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        int col = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < K; ++j) {
          if (j < F) {
            const int pq = readlane_i(vpq, j);
            const bool in = my[i] != j && !(my[i] > j && my[i] < F);
            if (in && sp[j][i] == rn[i].m1 && (pq & 0x1fff) < col) {
              col = pq & 0x1fff; rn[i].code = 2 * j; av[i] = xv[j][i];
            }
            if (in && sq[j][i] == rn[i].m1 && (pq >> 13) < col) {
              col = pq >> 13; rn[i].code = 2 * j + 1; av[i] = yv[j][i];
            }
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      const int pq = __shfl(vpq, rn[i].code >> 1);
      const int col = rn[i].code & 1 ? pq >> 13 : pq & 0x1fff;
      const bool moved = my[i] >= 0 && my[i] < F;
      if (ex.T + i * ex.GT < n) {
        if (moved) {
          dk[i] = dc[i];
          tk[i] = (int)(rot + my[i] + 1);
        }
        const bool up = row_refresh(bs[i], ba[i], bu[i], bst[i], moved, hs[i] < F, rn[i], col);
        bv[i] = up ? av[i] : bv[i];
      }
    }
    if (lane < F) {
      const int p = vpq & 0x1fff, q = vpq >> 13;
      ex.set_diag(p, q, vnp, vnq, (int)(rot + lane + 1));
      if (ex.first_wave()) d.log[rot - log_base + lane] = RotEntry{p, q, vc, vsn};
    }
    rot += F;
    kmax = min(K, F + 1 + (F == kk ? 1 : 0));
    lap(5);
  }

  // ---- write the state back (a later launch may resume from it)
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    const int k = ex.T + i * ex.GT;
    if (k < n) {
      d.diag[k] = dk[i]; d.bs[k] = bs[i]; d.ba[k] = ba[i]; d.bv[k] = bv[i]; d.bst[k] = bst[i];
      d.bu[k] = bu[i]; d.ts[k] = tk[i];
    }
  }
  if (prof && lane == 0)
    for (int k = 0; k < 6; ++k) d.prof[k] += tph[k];
  if (ex.first_wave() && lane == 0) {
    JCtl* ctl = d.ctl;
    ctl->rotations = rot;
    ctl->rescans += rescans;
    ctl->status = status;
    ctl->done = done;
    ctl->final_sel = wsel;
    ctl->final_cert = GAP ? wsel : -1.0;
    ctl->final_off = 0.0;
  }
  return done != 0;
}

}  // namespace je
