// One-sided Jacobi SVD (Algorithm 2) with the pivot scores of Sec. 3 evaluated on the Gram
// matrix A = B^T B (Sec. 2.1), including the relative score of Sec. 4.2.
//
// Layout: B (m x n, m >= n) is held row-major, Y[r][k] = b_rk with row stride ldy, so that
// the lanes computing a_pk for consecutive k read consecutive addresses while b_rp is a
// broadcast.  A is row-major n x n.  A is never rotated: every entry is the dot product of
// the current columns summed in index order (one lane per entry, no split of the sum), and
// after a rotation of columns p and q the rows p and q of A are recomputed.  With
// -ffp-contract=off every value is then a function of the input bits alone.
//
// One persistent launch runs the whole rotation sequence: one workgroup with B in LDS when it
// and the per-row state fit, several workgroups with a slice of B each above that, one
// workgroup with B in HBM beyond what 32 slices hold.  The last of these, per rotation:
//   argmax over the per-row best scores (each wave redundantly: no cross-wave exchange),
//   rotation of columns p, q of B and of rows p, q of the right factor V^T, barrier,
//   the dot products of rows p and q of A, barrier,
//   per-row cache refresh (Sec. 3.2), rows needing a full rescan queued in LDS, barrier,
//   full rescans, one wave per queued row, barrier.
#include <algorithm>

#include "device_common.h"
#include "jacobi_device.h"
#include "kernels.h"
#include "mw_exchange.h"
#include "svd_columns.h"

namespace je {

// Relative score of Sec. 4.2, (1/a_ii + 1/a_jj) L_ij: the sum of the relative shifts of the
// two eigenvalues of the 2 x 2 block.  It is invariant under scaling of the block, so the
// entries are first multiplied by the power of two that brings max(a_ii, a_jj) into
// [1/2, 1) (exact): a pair of tiny columns keeps a_ij^2 in range.  0 when a_ij == 0 or the
// scaled a_ij^2 underflows.
__device__ __forceinline__ double rel_score(double aii, double ajj, double aij) {
  if (aij == 0.0) return 0.0;
  int e;
  (void)frexp(fmax(aii, ajj), &e);
  const double x = ldexp(aii, -e), y = ldexp(ajj, -e), a = ldexp(aij, -e);
  const double l = gap_score(x, y, a);
  if (l == 0.0) return 0.0;
  return (1.0 / x + 1.0 / y) * l;
}

// PIV: 0 greedy |a_ij|, 1 gap L_ij (eq. (1)), 2 relative (Sec. 4.2)
template <int PIV>
__device__ __forceinline__ double svd_score(double aii, double ajj, double aij) {
  if constexpr (PIV == 0) return fabs(aij);
  else if constexpr (PIV == 1) return gap_score(aii, ajj, aij);
  else return rel_score(aii, ajj, aij);
}

// (score, index) maximum over the wave: larger score, then smaller index.  Every lane ends
// with the result.
__device__ __forceinline__ void wave_best(double& v, int& k) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ov = __shfl_xor(v, o);
    const int ok = __shfl_xor(k, o);
    if (ov > v || (ov == v && ok < k)) {
      v = ov;
      k = ok;
    }
  }
}

// ------------------------------------------------------------------ set-up kernels
// Y[r][k] = B[r + k ldb]; flags a non-finite entry.  32 x 32 tiles through LDS so that
// both the column-major reads and the row-major writes are coalesced.
__global__ __launch_bounds__(256) void k_svd_load(const double* __restrict__ B, int m, int n,
                                                  int ldb, double* __restrict__ Y, int ldy,
                                                  int* __restrict__ flag) {
  __shared__ double t[32][33];
  const int r0 = blockIdx.x * 32, k0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // ty in [0, 8)
  bool bad = false;
  for (int j = ty; j < 32; j += 8) {
    const int r = r0 + tx, k = k0 + j;
    if (r < m && k < n) {
      const double v = B[(size_t)k * ldb + r];
      bad |= !isfinite(v);
      t[j][tx] = v;
    }
  }
  if (bad) *flag = 1;
  __syncthreads();
  for (int j = ty; j < 32; j += 8) {
    const int r = r0 + j, k = k0 + tx;
    if (r < m && k < n) Y[(size_t)r * ldy + k] = t[tx][j];
  }
}

// A = B^T B: entry (i, j), i <= j, by one lane (j across the lanes of a row of 16), summed
// in index order, mirrored.
__global__ __launch_bounds__(256) void k_svd_gram(const double* __restrict__ Y, int ldy, int m,
                                                  int n, double* __restrict__ G, int ldg) {
  const int j = blockIdx.x * 16 + (threadIdx.x & 15);
  const int i = blockIdx.y * 16 + (threadIdx.x >> 4);
  if (i >= n || j >= n || i > j) return;
  double s = 0.0;
#pragma unroll 8
  for (int r = 0; r < m; ++r) s += Y[(size_t)r * ldy + i] * Y[(size_t)r * ldy + j];
  G[(size_t)i * ldg + j] = s;
  G[(size_t)j * ldg + i] = s;
}

// Best (score, column) of every row, one wave per row (smallest column on ties); also the
// diagonal of A.
template <int PIV>
__global__ __launch_bounds__(256) void k_svd_rowbest(const double* __restrict__ G, int ldg,
                                                     int n, double* __restrict__ best,
                                                     int* __restrict__ arg,
                                                     double* __restrict__ diag) {
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (k >= n) return;
  const double* gk = G + (size_t)k * ldg;
  const double akk = gk[k];
  double v = -1.0;
  int c = INT_MAX;
  for (int l = lane; l < n; l += 64) {
    if (l == k) continue;
    const double x = svd_score<PIV>(akk, G[(size_t)l * ldg + l], gk[l]);
    if (x > v) {
      v = x;
      c = l;
    }
  }
  wave_best(v, c);
  if (lane == 0) {
    best[k] = v;
    arg[k] = c == INT_MAX ? -1 : c;
    diag[k] = akk;
  }
}

// Z = Y Q (Z[r][k] = sum_i Y[r][i] Q[i][k], summed in index order): B times the
// preconditioner.
__global__ __launch_bounds__(256) void k_svd_rowmix(const double* __restrict__ Y, int ldy,
                                                    const double* __restrict__ Q, int ldq,
                                                    int m, int n, double* __restrict__ Z,
                                                    int ldz) {
  const int r = blockIdx.y;
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  const double* yr = Y + (size_t)r * ldy;
  double s = 0.0;
  for (int i = 0; i < n; ++i) s += yr[i] * Q[(size_t)i * ldq + k];
  Z[(size_t)r * ldz + k] = s;
}

// Vt = Q^T.
__global__ __launch_bounds__(256) void k_svd_transpose(const double* __restrict__ Q, int ldq,
                                                       int n, double* __restrict__ Vt,
                                                       int ldv) {
  const int k = blockIdx.y;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256)
    Vt[(size_t)k * ldv + i] = Q[(size_t)i * ldq + k];
}

// Yc[k][r] = Y[r][k] (32 x 32 tiles through LDS): B column by column.
__global__ __launch_bounds__(256) void k_svd_columns(const double* __restrict__ Y, int ldy, int m,
                                                     int n, double* __restrict__ Yc, int ldc) {
  __shared__ double t[32][33];
  const int r0 = blockIdx.x * 32, k0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int j = ty; j < 32; j += 8)
    if (r0 + j < m && k0 + tx < n) t[j][tx] = Y[(size_t)(r0 + j) * ldy + k0 + tx];
  __syncthreads();
  for (int j = ty; j < 32; j += 8)
    if (k0 + j < n && r0 + tx < m) Yc[(size_t)(k0 + j) * ldc + r0 + tx] = t[tx][j];
}

// ------------------------------------------------------------------ the rotation sequence
// Barrier for phases that communicate through LDS only: waits for this wave's LDS accesses,
// not for its stores to device memory (which no other wave reads before the kernel ends).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Wave-uniform (score, index) maximum, larger score then smaller index, of per-lane
// candidates (v < 0: none).  Returns false when no lane has a candidate.
__device__ __forceinline__ bool wave_best_fast(double& v, int& k) {
  const int w = wave_argmax_lane(v, k);
  if (w < 0) return false;
  v = readlane_d(v, w);
  k = readlane_i(k, w);
  return true;
}

// Bytes of dynamic LDS of the resident mode: B by columns with an odd stride (the lanes' reads of
// their own columns then fall in distinct banks), zeros, and rows p, q and the diagonal of A.
constexpr int kSvdResMaxN = 128, kSvdResPad = 24;
// Up to this n the kernel stores the entries of A that a rotation changes (KEEP); above it A is
// formed once more at the end.  Few columns take few rotations, and forming A again is m dependent
// sums of 22 ns: 4060 x 2 0.53 ms a call with it, 0.42 without (1000 x 8 1.48 and 1.45).
constexpr int kSvdResKeepN = 8;
// the rotated columns once more, with zeros up to the reads ahead of the last term
__host__ __device__ __forceinline__ int svd_col_len(int m) { return ((m + 15) & ~15) + 8; }
__host__ __device__ __forceinline__ int svd_lds_ld(int m) { return m | 1; }
__host__ __device__ __forceinline__ size_t svd_lds_bytes(int m, int n) {
  return 8 * ((size_t)n * svd_lds_ld(m) + kSvdResPad + 2 * (size_t)svd_col_len(m) +
              3 * kSvdResMaxN + 1);
}

struct SvdBestAt {
  double s, a;  // score (-1: none) and entry
  int c;        // column
};

struct SvdRow {
  SvdBestAt x, y;  // best and second best
  double u;        // bound of the others
};

__device__ __forceinline__ bool svd_before(const SvdBestAt& a, const SvdBestAt& b) {
  return a.s > b.s || (a.s == b.s && a.c < b.c);
}

__device__ __forceinline__ SvdBestAt svd_pick(bool w, const SvdBestAt& a, const SvdBestAt& b) {
  return SvdBestAt{w ? a.s : b.s, w ? a.a : b.a, w ? a.c : b.c};
}

__device__ __forceinline__ SvdBestAt svd_none() { return SvdBestAt{-1.0, 0.0, INT_MAX}; }

// The best two of two ordered pairs; the bound takes the other two.
__device__ __forceinline__ void svd_row_merge(SvdRow& r, const SvdBestAt& x, const SvdBestAt& y) {
  const bool w = svd_before(x, r.x);
  const SvdBestAt l = svd_pick(w, r.x, x), sw = svd_pick(w, y, r.y);
  const double o = w ? r.y.s : y.s;
  const bool v = svd_before(l, sw);
  r.x = svd_pick(w, x, r.x);
  r.y = svd_pick(v, l, sw);
  r.u = fmax(fmax(r.u, o), v ? sw.s : l.s);
}

// The best two of one wave's entries of rows p and q (score, column k, entry per lane) and a
// bound of the rest, the two rows' chains interleaved: out[row] = s, a, s', a', bound, c | c' << 32.
__device__ __forceinline__ void svd_search2(double ep, double vp, double eq, double vq, int k,
                                            double (*out)[6], int lane) {
  int a = key32(ep), b = key32(eq);
  auto max2 = [](int x, int y, int& mx, int& my) {
    x = max(x, dpp_i<0xB1>(x)); y = max(y, dpp_i<0xB1>(y));
    x = max(x, dpp_i<0x4E>(x)); y = max(y, dpp_i<0x4E>(y));
    x = max(x, dpp_i<0x141>(x)); y = max(y, dpp_i<0x141>(y));
    x = max(x, dpp_i<0x140>(x)); y = max(y, dpp_i<0x140>(y));
    auto rows = [](int m) {
      return max(max(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16)),
                 max(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
    };
    mx = rows(x);
    my = rows(y);
  };
  if (lane < 2) {
    out[lane][0] = out[lane][2] = -1.0;
    out[lane][1] = out[lane][3] = 0.0;
    reinterpret_cast<int*>(&out[lane][5])[0] = reinterpret_cast<int*>(&out[lane][5])[1] = INT_MAX;
  }
  int ma, mb;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    max2(a, b, ma, mb);
    const int la = argmax_finish(ep, k, a, ma), lb = argmax_finish(eq, k, b, mb);
    if (lane == la) {
      out[0][2 * e] = ep;
      out[0][2 * e + 1] = vp;
      reinterpret_cast<int*>(&out[0][5])[e] = k;
    }
    if (lane == lb) {
      out[1][2 * e] = eq;
      out[1][2 * e + 1] = vq;
      reinterpret_cast<int*>(&out[1][5])[e] = k;
    }
    a = lane == la ? -1 : a;
    b = lane == lb ? -1 : b;
  }
  max2(a, b, ma, mb);
  if (lane < 2) out[lane][4] = key_ub(lane ? mb : ma);
}

// Resident mode, n <= 128: B stays in LDS for the whole run.  The bound is the chain of one
// rotation: the pick, its parameters, the dot products of rows p and q of A, their scores.
//
// Dot products: lane k forms a_pk, lane 128 + k a_qk, in index order, from the lanes' own columns
// and a copy of the rotated one, in two blocks of 8 terms in turn, each read while the other is
// summed (13.3 ns a term; 24.7 with one block read, then summed; 17.6 with the rotated column
// across the lanes, handed round by v_readlane).  The limit is one wave's LDS reads, 16 bytes a
// lane in 21 cycles.  A itself is not kept: its entries are needed where they change and in the
// rare rescan, which forms them again (same products, same order, same bits); of up to kSvdResKeepN
// columns they are stored as they change.
//
// Caches: lane k < 128 owns row k's: its exact best (score, column, entry), the second best, and a
// bound of the others.  A row whose best moved down takes its second best or a new entry, where
// that lies above the bound, and is rescanned before the next selection otherwise (Hilbert
// matrix's factor of order 100, relative score: 0.93 rows per rotation lose their best, 0.02 are
// rescanned).  Lanes 128 .. 255 search the new rows p and q while the others select and rotate;
// until then those two rows' caches hold the pair (p, q) alone, as every other new pair is in
// the other row's cache.
//
// Measured, per rotation, before (A in LDS, a rescan for every best that moved down) and now:
// Hilbert factor of order 100 4.70 -> 3.73 us (dot products 1.2, parameters and columns 0.75,
// scores 0.7, caches 0.3, selection 0.3, rescans 0.2), 130 x 100 5.0 -> 4.4, 500 x 30 10.3 -> 8.9,
// 130 x 128 (on several workgroups before) 7.1 -> 4.3.  Dot products of 16 terms at a time, with
// up to 15 zeros at the end, took 4.0, 4.6, 9.5 and 4.5, and 33 x 16 6% longer than before.
template <int PIV, bool KEEP>
__global__ __launch_bounds__(256) void k_svd_res(const SDesc d) {
  constexpr int NT = 256, kB = 8;
  extern __shared__ __attribute__((aligned(16))) double smem[];
  __shared__ __attribute__((aligned(16))) double s_slot[2][4], s_pq[2][2][6], s_cs[2];
  __shared__ int s_list[kSvdResMaxN], s_cnt, s_resc;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int half = tid >> 7, k = tid & (kSvdResMaxN - 1);
  const int n = d.n, m = d.m, ldc = svd_lds_ld(m);
  const size_t ldv = d.ldv;
  const int cl = svd_col_len(m);
  double* colp = smem;
  double* colq = colp + cl;
  double* Yc = colq + cl;  // column k of B from Yc + k ldc
  double* rowp = Yc + (size_t)n * ldc + kSvdResPad;
  double* rowq = rowp + kSvdResMaxN;
  double* diag = rowq + kSvdResMaxN;
  for (int i = tid; i < n * ldc; i += NT) {
    const int r = i / n, c = i - r * n;
    Yc[c * ldc + r] = r < m ? d.Y[(size_t)r * d.ldy + c] : 0.0;
  }
  for (int i = tid; i < 2 * cl; i += NT) colp[i] = 0.0;
  if (tid < n) diag[tid] = d.diag[tid];
  if (tid < kSvdResPad) Yc[(size_t)n * ldc + tid] = 0.0;
  if (tid == 0) {
    s_cnt = 0;
    s_resc = 0;
  }
  __syncthreads();
  const bool act = k < n;
  const double* mine = Yc + (act ? k : 0) * ldc;
  // sum_i u_i z_i in index order, z this lane's column, read a block of 8 ahead; the terms that
  // fill up the last 8 have u_i = 0 and a finite z_i (the next column's, or the zeros behind
  // the last)
  auto dot = [&](const double* u) -> double {
    double x = 0.0, u0[kB], z0[kB], u1[kB], z1[kB];
#pragma unroll
    for (int e = 0; e < kB; ++e) u0[e] = u[e];
#pragma unroll
    for (int e = 0; e < kB; ++e) z0[e] = mine[e];
    int i = 0;
#pragma unroll 1
    for (; i + kB < m; i += 2 * kB) {
#pragma unroll
      for (int e = 0; e < kB; ++e) u1[e] = u[i + kB + e];
#pragma unroll
      for (int e = 0; e < kB; ++e) z1[e] = mine[i + kB + e];
#pragma unroll
      for (int e = 0; e < kB; ++e) x += u0[e] * z0[e];
#pragma unroll
      for (int e = 0; e < kB; ++e) u0[e] = u[i + 2 * kB + e];
#pragma unroll
      for (int e = 0; e < kB; ++e) z0[e] = mine[i + 2 * kB + e];
#pragma unroll
      for (int e = 0; e < kB; ++e) x += u1[e] * z1[e];
    }
    if (i < m) {
#pragma unroll
      for (int e = 0; e < kB; ++e) x += u0[e] * z0[e];
    }
    return x;
  };
  auto uni = [](int v) -> int { return __builtin_amdgcn_readfirstlane(v); };
  auto score = [&](double x, double y, double a) -> double {
    const double s = svd_score<PIV>(x, y, a);
    return s >= 0.0 ? s : -1.0;
  };

  double dk = act ? d.diag[k] : 0.0;
  SvdRow row{svd_none(), svd_none(), -1.0};
  if (half == 0 && act) {
    row.x.s = d.best[k];
    row.x.c = d.arg[k];
    if (row.x.c >= 0) row.x.a = d.G[(size_t)k * d.ldg + row.x.c];
    row.u = row.x.s;  // the others are no better
  }
  // rows whose search is under way in lanes 128 .. 255: their scores, and the lanes that wait
  int pend = -1, resc = 0;  // 0 / 1: this lane's row is row p / q of the last rotation
  double ep = -1.0, eq = -1.0, vp = 0.0, vq = 0.0;
  auto search = [&]() { svd_search2(ep, vp, eq, vq, k, s_pq[wv & 1], lane); };
  // the row's second best and bound after a rotation, from its caches before (x0, y0) and the
  // new entries
  SvdBestAt hi = svd_none(), lo = svd_none(), x0 = svd_none(), y0 = svd_none();
  bool lost = false, won = false;
  auto settle = [&]() {
    const SvdBestAt y1 = svd_pick(lost, svd_none(), y0);
    const SvdBestAt l = svd_pick(won, x0, hi), sw = svd_pick(won, lo, y1);
    const bool v = l.s > sw.s;
    row.y = svd_pick(v, l, sw);
    row.u = fmax(fmax(row.u, won ? y1.s : lo.s), v ? sw.s : l.s);
    if (!(row.y.s > row.u)) row.y = svd_none();
  };
  // a second best that another entry may equal is not kept
  auto trim = [&]() {
    const bool keep = row.y.s > row.u;
    row.y = svd_pick(keep, row.y, svd_none());
  };
  auto found = [&]() {
    if (pend >= 0) {
      const double* o0 = s_pq[0][pend];
      const double* o1 = s_pq[1][pend];
      const int* c0 = reinterpret_cast<const int*>(o0 + 5);
      const int* c1 = reinterpret_cast<const int*>(o1 + 5);
      row = SvdRow{{o0[0], o0[1], c0[0]}, {o0[2], o0[3], c0[1]}, fmax(o0[4], o1[4])};
      svd_row_merge(row, {o1[0], o1[1], c1[0]}, {o1[2], o1[3], c1[1]});
      trim();
      pend = -1;
    }
  };
  long long rot = 0;
  int status = ST_OK;
  double vsel = -1.0;
  bool moving = false;  // a search is pending
  for (;;) {
    // ---- the best pair; rows without a known best are rescanned first
    if (half == 0) {
      const int w = wave_argmax_lane(row.x.s, k);
      if (lane == max(w, 0)) {
        s_slot[wv][0] = w >= 0 ? row.x.s : -1.0;
        s_slot[wv][1] = row.x.a;
        s_slot[wv][2] = __longlong_as_double((long long)(k | row.x.c << 16));
      }
    }
    lds_barrier();
    const double v0 = s_slot[0][0], a0 = s_slot[0][1], v1 = s_slot[1][0], a1 = s_slot[1][1];
    const int rc0 = (int)__double_as_longlong(s_slot[0][2]);
    const int rc1 = (int)__double_as_longlong(s_slot[1][2]);
    const int cnt = uni(s_cnt);
    if (cnt > 0) {
      if (moving) settle();
      if (moving && half) search();
      lds_barrier();
      found();
      moving = false;
      for (int e = 0; e < cnt; e += 2) {
        const int r0 = uni(s_list[e]), r1 = uni(s_list[min(e + 1, cnt - 1)]);
        for (int i = tid; i < m; i += NT) {
          colp[i] = Yc[r0 * ldc + i];
          colq[i] = Yc[r1 * ldc + i];
        }
        lds_barrier();
        const double x = dot(half ? colq : colp);
        (half ? rowq : rowp)[k] = x;
        lds_barrier();
        vp = rowp[k];
        vq = rowq[k];
        ep = act && k != r0 ? score(dk, diag[r0], vp) : -1.0;
        eq = act && k != r1 ? score(dk, diag[r1], vq) : -1.0;
        if (half) search();
        if (half == 0 && (k == r0 || k == r1)) pend = k == r0 ? 0 : 1;
        lds_barrier();
        found();
      }
      if (tid == 0) s_cnt = 0;
      continue;
    }
    const bool w = v1 > v0;
    const double v = w ? v1 : v0, apq = w ? a1 : a0;
    const int rc = uni(w ? rc1 : rc0);
    vsel = v;
    if (n < 2 || v <= d.thr) break;
    if (rot >= d.maxrot) {
      status = ST_MAXROT;
      break;
    }
    if (apq == 0.0) {
      status = ST_STALL;
      break;
    }
    const int p = min(rc & 0xffff, rc >> 16), q = max(rc & 0xffff, rc >> 16);
    // ---- columns p and q of B; rows p and q of V^T, whose entries keep their lane for the
    // whole run, are loaded now and stored after the dot products
    const bool hv = d.Vt != nullptr && half && act;
    double vu = 0.0, vw = 0.0;
    if (hv) {
      vu = d.Vt[(size_t)p * ldv + k];
      vw = d.Vt[(size_t)q * ldv + k];
    }
    if (half && moving) search();
    if (wv * 64 < m) {
      double* yp = Yc + p * ldc;
      double* yq = Yc + q * ldc;
      const double u0 = tid < m ? yp[tid] : 0.0, x0 = tid < m ? yq[tid] : 0.0;
      double t, c, s;
      rot_params<double>(diag[p], diag[q], apq, t, c, s);
      if (moving) settle();
      if (tid < m) {
        yp[tid] = colp[tid] = c * u0 + s * x0;
        yq[tid] = colq[tid] = c * x0 - s * u0;
      }
      for (int i = tid + NT; i < m; i += NT) {
        const double u = yp[i], x = yq[i];
        yp[i] = colp[i] = c * u + s * x;
        yq[i] = colq[i] = c * x - s * u;
      }
      if (tid == 0) {
        s_cs[0] = c;
        s_cs[1] = s;
        if (d.plog && rot < d.logcap) {
          d.plog[2 * rot] = p;
          d.plog[2 * rot + 1] = q;
        }
      }
    }
    ++rot;
    lds_barrier();
    // ---- rows p and q of A
    const bool own = k == p || k == q;
    const double x = dot(half ? colq : colp);
    (half ? rowq : rowp)[k] = x;
    if (hv) {
      const double c = s_cs[0], s = s_cs[1];
      d.Vt[(size_t)p * ldv + k] = c * vu + s * vw;
      d.Vt[(size_t)q * ldv + k] = c * vw - s * vu;
    }
    lds_barrier();
    // ---- scores and caches (a_pq is row p's, the same bits as row q's)
    found();
    const double app = rowp[p], aqq = rowq[q];
    vp = rowp[k];
    vq = k == p ? rowp[q] : rowq[k];
    dk = k == p ? app : (k == q ? aqq : dk);
    ep = act && k != p ? score(dk, app, vp) : -1.0;
    eq = act && k != q ? score(dk, aqq, vq) : -1.0;
    moving = true;
    if constexpr (KEEP) {
      if (half == 0 && act) {
        d.G[(size_t)p * d.ldg + k] = d.G[(size_t)k * d.ldg + p] = vp;
        d.G[(size_t)q * d.ldg + k] = d.G[(size_t)k * d.ldg + q] = vq;
      }
    }
    if (tid == NT - 1) {
      diag[p] = app;
      diag[q] = aqq;
    }
    // the best of this lane's row now; what follows the best waits for settle()
    const bool hit = row.x.c == p || row.x.c == q, hit2 = row.y.c == p || row.y.c == q;
    const bool qf = eq > ep;
    hi = SvdBestAt{qf ? eq : ep, qf ? vq : vp, qf ? q : p};
    lo = SvdBestAt{qf ? ep : eq, qf ? vp : vq, qf ? p : q};
    lost = hit && !own;
    y0 = svd_pick(hit2 || own, svd_none(), row.y);
    x0 = svd_pick(own, svd_none(), svd_pick(hit, y0, row.x));
    if (half == 0 && !own && hit && !(hi.s > row.x.s || (hi.s == row.x.s && hi.c <= row.x.c))) ++resc;
    if (own) {
      pend = k == p ? 0 : 1;
      hi = SvdBestAt{k == p ? eq : ep, k == p ? vq : vp, k == p ? q : p};
      lo = svd_none();
      row.u = -1.0;
    }
    won = svd_before(hi, x0);
    row.x = svd_pick(won, hi, x0);
    // the best is exact if it was before, or is above every entry not held here
    if (half == 0 && act && lost && !(row.x.s > row.u)) s_list[atomicAdd(&s_cnt, 1)] = k;
  }
  __syncthreads();
  for (int i = tid; i < m * n; i += NT) {
    const int r = i / n, c = i - r * n;
    d.Y[(size_t)r * d.ldy + c] = Yc[c * ldc + r];
  }
  if (resc) atomicAdd(&s_resc, resc);
  __syncthreads();
  if (tid == 0) {
    d.ctl->rotations = rot;
    d.ctl->rescans = s_resc;
    d.ctl->status = status;
    d.ctl->done = 1;
    d.ctl->final_sel = vsel;
  }
}

// HBM mode (B too large for LDS): B, A and the per-row state in device memory, the rescan
// queue in LDS; the same steps with full barriers.
template <int PIV, int NT>
__global__ __launch_bounds__(NT) void k_svd1(const SDesc d) {
  constexpr int NW = NT / 64;
  extern __shared__ int list[];
  __shared__ int s_cnt, s_resc;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = d.n, m = d.m;
  double* __restrict__ G = d.G;
  double* __restrict__ Y = d.Y;
  double* __restrict__ best = d.best;
  double* __restrict__ diag = d.diag;
  double* __restrict__ rowp = d.rowp;
  double* __restrict__ rowq = d.rowq;
  int* __restrict__ arg = d.arg;
  const size_t ldg = d.ldg, ldv = d.ldv, ldy = d.ldy;
  if (tid == 0) s_resc = 0;
  __syncthreads();
  long long rot = 0;
  int status = ST_OK;
  double vsel = -1.0;
  for (;;) {
    double v = -1.0;
    int r = INT_MAX;
    for (int k = lane; k < n; k += 64) {
      const double x = best[k];
      if (x > v) {
        v = x;
        r = k;
      }
    }
    if (!wave_best_fast(v, r)) v = -1.0;
    vsel = v;
    if (n < 2 || v <= d.thr) break;
    if (rot >= d.maxrot) {
      status = ST_MAXROT;
      break;
    }
    const int a = arg[r];
    const int p = min(r, a), q = max(r, a);
    const double apq = G[(size_t)p * ldg + q];
    if (apq == 0.0) {
      status = ST_STALL;
      break;
    }
    double t, c, s;
    rot_params<double>(diag[p], diag[q], apq, t, c, s);
    for (int i = tid; i < m; i += NT) {
      double* yi = Y + (size_t)i * ldy;
      const double u = yi[p], w = yi[q];
      yi[p] = c * u + s * w;
      yi[q] = c * w - s * u;
    }
    if (d.Vt) {
      double* vp = d.Vt + (size_t)p * ldv;
      double* vq = d.Vt + (size_t)q * ldv;
      for (int i = tid; i < n; i += NT) {
        const double u = vp[i], w = vq[i];
        vp[i] = c * u + s * w;
        vq[i] = c * w - s * u;
      }
    }
    if (tid == 0) {
      if (d.plog && rot < d.logcap) {
        d.plog[2 * rot] = p;
        d.plog[2 * rot + 1] = q;
      }
      s_cnt = 0;
    }
    ++rot;
    __syncthreads();
    // both dot products of column k in one pass over B
    for (int k = tid; k < n; k += NT) {
      constexpr int kB = 16;
      double xp = 0.0, xq = 0.0;
      int i = 0;
      for (; i + kB <= m; i += kB) {
        double u[kB], w[kB], z[kB];
#pragma unroll
        for (int j = 0; j < kB; ++j) {
          const double* yi = Y + (size_t)(i + j) * ldy;
          u[j] = yi[p];
          w[j] = yi[q];
          z[j] = yi[k];
        }
#pragma unroll
        for (int j = 0; j < kB; ++j) {
          xp += u[j] * z[j];
          xq += w[j] * z[j];
        }
      }
      for (; i < m; ++i) {
        const double* yi = Y + (size_t)i * ldy;
        const double yk = yi[k];
        xp += yi[p] * yk;
        xq += yi[q] * yk;
      }
      rowp[k] = xp;
      rowq[k] = xq;
      G[(size_t)p * ldg + k] = xp;
      G[(size_t)k * ldg + p] = xp;
      G[(size_t)q * ldg + k] = xq;
      G[(size_t)k * ldg + q] = xq;
      if (k == p) diag[p] = xp;
      if (k == q) diag[q] = xq;
    }
    __syncthreads();
    const double app = diag[p], aqq = diag[q];
    for (int k = tid; k < n; k += NT) {
      if (k == p || k == q) {
        list[atomicAdd(&s_cnt, 1)] = k;
        continue;
      }
      const double akk = diag[k];
      const double sp = svd_score<PIV>(akk, app, rowp[k]);
      const double sq = svd_score<PIV>(akk, aqq, rowq[k]);
      double b = best[k];
      int ak = arg[k];
      if (ak == p || ak == q) {
        double x = sp;
        int col = p;
        if (sq > x) {
          x = sq;
          col = q;
        }
        if (x > b || (x == b && col <= ak)) {
          best[k] = x;
          arg[k] = col;
        } else {
          list[atomicAdd(&s_cnt, 1)] = k;
          atomicAdd(&s_resc, 1);
        }
      } else {
        if (sp > b || (sp == b && p < ak)) {
          b = sp;
          ak = p;
        }
        if (sq > b || (sq == b && q < ak)) {
          b = sq;
          ak = q;
        }
        best[k] = b;
        arg[k] = ak;
      }
    }
    __syncthreads();
    const int cnt = s_cnt;
    for (int e = wv; e < cnt; e += NW) {
      const int k = list[e];
      const double* gk = G + (size_t)k * ldg;
      const double akk = diag[k];
      double bv = -1.0;
      int bc = INT_MAX;
      for (int l = lane; l < n; l += 64) {
        if (l == k) continue;
        const double x = svd_score<PIV>(akk, diag[l], gk[l]);
        if (x > bv) {
          bv = x;
          bc = l;
        }
      }
      wave_best_fast(bv, bc);
      if (lane == 0) {
        best[k] = bv;
        arg[k] = bc;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    d.ctl->rotations = rot;
    d.ctl->rescans = s_resc;
    d.ctl->status = status;
    d.ctl->done = 1;
    d.ctl->final_sel = vsel;
  }
}

// ------------------------------------------------------------------ several workgroups
// B too large for one LDS: G workgroups on one XCD hold c columns of it each, in LDS for the
// whole run.  Column-major copies of B in device memory carry the columns between them: two of
// each column (svd_columns.h), since in a rotation the owners store the new columns p, q while
// other workgroups may still load the old ones.
// Per rotation every workgroup
//   loads the current copies of columns p, q (L2), rotates them into LDS (the owners also store
//   them over the other copies);
//   forms the dot products of its columns with the new p and q, one lane each in index order,
//   and those of p and q with themselves;
//   stores its entries of A (rows and columns p, q), refreshes the caches of its rows, rescans
//   those whose best moved down, and finds its part of the new rows' bests;
//   exchanges its best row and those two, after which all hold the same winner.
// Bound: the dot products (dot_in_order), then the exchange (0.6 us) and the L2 reads of the
// columns and of the rows rescanned.  One workgroup alone read all of B from L2 at 22 GB/s per
// rotation: 1024 x 512 186 -> 15 us per rotation, 300 x 260 38.8 -> 8.9, 130 x 129 13.4 -> 6.8.
constexpr int kSvdMwThreads = 256;
constexpr int kSvdMwWords = 9;  // three candidates: score, entry, row << 32 | column

// Row stride of the LDS columns: even (16-byte loads) and 4 banks apart from column to column
// (no more than even for two or three columns, which meet in few banks in any case: 4066 x 3
// still fits).
__host__ __device__ __forceinline__ int svd_mw_stride(int m, int c) {
  return c < 4 ? (m + 1) & ~1 : (m + 31) / 32 * 32 + 2;
}

__host__ __device__ __forceinline__ size_t svd_mw_lds(int m, int n, int c) {
  return 8 * ((size_t)(c + 2) * svd_mw_stride(m, c) + n + 4 * (size_t)c) + 8 * (size_t)c;
}

// sum_i u_i y_i in index order, the operands of 8 terms in flight ahead of the sums.  What bounds
// it is the LDS return path of the one wave (both factors, 16 bytes a lane in 21 cycles; the
// chain of products and sums alone takes 10 cycles a step).  Two blocks in turn, each loaded while
// the other is summed, measured 14.6 us per rotation at 1024 x 512; one block of 16 whose
// operands and products move up by copies 16.9; handing u round a row of lanes on the DPP
// network instead of reading it is slower again (1009 x 33: 18.7 against 17.2).
__device__ __forceinline__ double dot_in_order(const double* u, const double* y, int m) {
  constexpr int kB = 8;
  double x = 0.0;
  int i = 0;
  if (m >= 2 * kB) {
    double2 a[kB / 2], b[kB / 2], v[kB / 2], w[kB / 2];
    auto load = [&](double2* p, double2* q, int at) {
#pragma unroll
      for (int e = 0; e < kB / 2; ++e) p[e] = *reinterpret_cast<const double2*>(u + at + 2 * e);
#pragma unroll
      for (int e = 0; e < kB / 2; ++e) q[e] = *reinterpret_cast<const double2*>(y + at + 2 * e);
    };
    auto sum = [&](const double2* p, const double2* q) {
#pragma unroll
      for (int e = 0; e < kB / 2; ++e) {
        x += p[e].x * q[e].x;
        x += p[e].y * q[e].y;
      }
    };
    load(a, b, 0);
#pragma unroll 1
    for (; i + 2 * kB <= m; i += 2 * kB) {
      load(v, w, i + kB);
      sum(a, b);
      load(a, b, i + 3 * kB <= m ? i + 2 * kB : 0);
      sum(v, w);
    }
  }
  for (; i < m; ++i) x += u[i] * y[i];
  return x;
}

// (score, column) maximum of a wave's lanes with its entry, every lane the result.
struct SvdBest {
  double v, a;
  int c;
};

__device__ __forceinline__ SvdBest wave_svd_best(double v, int c, double a) {
  const int w = wave_argmax_lane(v, c);
  if (w < 0) return SvdBest{-1.0, 0.0, INT_MAX};
  return SvdBest{readlane_d(v, w), readlane_d(a, w), readlane_i(c, w)};
}

template <int PIV>
__global__ __launch_bounds__(kSvdMwThreads) void k_svd_mw(const SDesc d, MwCtl* mc, double* xb,
                                                          double* Yc, int ldc, int G, int c) {
  if (blockIdx.x % kMwStride) return;
  const int g = blockIdx.x / kMwStride;
  if (g >= G) return;
  constexpr int NT = kSvdMwThreads, NW = NT / 64;
  extern __shared__ __align__(16) double smem[];
  __shared__ int s_cnt, s_ok, s_rc[3];
  __shared__ double s_best[3], s_val[3], s_new[2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = d.n, m = d.m, S = svd_mw_stride(m, c);
  const int k0 = g * c, nk = min(c, n - k0);
  const size_t ldg = d.ldg, ldv = d.ldv;
  double* Ys = smem;
  double* colp = Ys + (size_t)c * S;
  double* colq = colp + S;
  double* diag = colq + S;
  double* best = diag + n;
  double* val = best + c;
  double* xp = val + c;
  double* xq = xp + c;
  int* arg = (int*)(xq + c);
  int* list = arg + c;

  int round = 1;
  if (wv == 0) {
    const bool ok = mw_start(mc, G, g, round);
    if (lane == 0) s_ok = ok;
  }
  __syncthreads();
  if (!s_ok) return;

  for (int k = 0; k < nk; ++k)
    for (int i = tid; i < m; i += NT) Ys[(size_t)k * S + i] = Yc[(size_t)(k0 + k) * ldc + i];
  for (int k = tid; k < n; k += NT) diag[k] = d.diag[k];
  for (int k = tid; k < nk; k += NT) {
    best[k] = d.best[k0 + k];
    const int a = d.arg[k0 + k];
    arg[k] = a;
    val[k] = a >= 0 ? d.G[(size_t)(k0 + k) * ldg + a] : 0.0;
  }
  if (tid == 0) s_cnt = 0;
  __syncthreads();

  long long rot = 0, resc = 0;
  int status = ST_OK, p = -1, q = -1;
  double vsel = -1.0;
  bool failed = false;
  unsigned ver = 0;  // versions of the columns (svd_columns.h), the same in every wave
  auto version = [&](int k) -> unsigned {
    return (unsigned)readlane_i((int)ver, svd_version_lane(k)) & svd_version_bit(k);
  };
  // this lane's part of the new rows p and q (wave 0)
  double vp = -1.0, ap = 0.0, vq = -1.0, aq = 0.0;
  int cp = INT_MAX, cq = INT_MAX;
  for (;;) {
    // ---- exchange: wave 0 publishes and reads, the others wait
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);  // this wave's stores have reached L2
    __syncthreads();
    ++round;
    if (wv == 0) {
      double v = -1.0, a = 0.0;
      int r = INT_MAX, rc = 0;
      for (int k = lane; k < nk; k += 64) {
        if (k0 + k == p || k0 + k == q) continue;
        if (best[k] > v) { v = best[k]; r = k0 + k; rc = arg[k]; a = val[k]; }
      }
      const int w = wave_argmax_lane(v, r);
      const SvdBest bp = wave_svd_best(vp, cp, ap), bq = wave_svd_best(vq, cq, aq);
      double* my = xb + (size_t)((round & 1) * G + g) * kSvdMwWords;
      if (lane == (w < 0 ? 0 : w)) {
        st_ag(my, w < 0 ? -1.0 : v);
        st_ag(my + 1, a);
        st_ag(my + 2, __longlong_as_double((long long)r << 32 | (unsigned)rc));
      }
      if (lane == 0) {
        st_ag(my + 3, bp.v);
        st_ag(my + 4, bp.a);
        st_ag(my + 5, __longlong_as_double((long long)bp.c));
        st_ag(my + 6, bq.v);
        st_ag(my + 7, bq.a);
        st_ag(my + 8, __longlong_as_double((long long)bq.c));
      }
      const bool ok = mw_sync(mc, G, round);
      double s1 = -1.0, a1 = 0.0, s2 = -1.0, a2 = 0.0, s3 = -1.0, a3 = 0.0;
      long long i1 = 0, i2 = 0, i3 = 0;
      if (ok && lane < G) {
        const double* sl = xb + (size_t)((round & 1) * G + lane) * kSvdMwWords;
        s1 = ld_ag(sl); a1 = ld_ag(sl + 1); i1 = __double_as_longlong(ld_ag(sl + 2));
        s2 = ld_ag(sl + 3); a2 = ld_ag(sl + 4); i2 = __double_as_longlong(ld_ag(sl + 5));
        s3 = ld_ag(sl + 6); a3 = ld_ag(sl + 7); i3 = __double_as_longlong(ld_ag(sl + 8));
      }
      const int r1 = (int)(i1 >> 32), c1 = (int)i1;
      const int w1 = wave_argmax_lane(s1, r1);
      double bv = -1.0, ba = 0.0;
      int br = INT_MAX, bc = 0;
      if (w1 >= 0) {
        bv = readlane_d(s1, w1); ba = readlane_d(a1, w1);
        br = readlane_i(r1, w1); bc = readlane_i(c1, w1);
      }
      const SvdBest np_ = wave_svd_best(s2, (int)i2, a2), nq_ = wave_svd_best(s3, (int)i3, a3);
      // rows p and q of the last rotation (p < q): ties to the smaller row
      if (p >= 0) {
        if (np_.v > bv || (np_.v == bv && p < br)) { bv = np_.v; ba = np_.a; br = p; bc = np_.c; }
        if (nq_.v > bv || (nq_.v == bv && q < br)) { bv = nq_.v; ba = nq_.a; br = q; bc = nq_.c; }
      }
      if (lane == 0) {
        s_ok = ok;
        s_best[0] = bv; s_val[0] = ba; s_rc[0] = br; s_rc[1] = bc;
        if (p >= k0 && p < k0 + nk) { best[p - k0] = np_.v; arg[p - k0] = np_.c; val[p - k0] = np_.a; }
        if (q >= k0 && q < k0 + nk) { best[q - k0] = nq_.v; arg[q - k0] = nq_.c; val[q - k0] = nq_.a; }
      }
    }
    __syncthreads();
    if (!s_ok) { failed = true; break; }
    vsel = s_best[0];
    if (n < 2 || vsel <= d.thr) break;
    if (rot >= d.maxrot) { status = ST_MAXROT; break; }
    const double apq = s_val[0];
    if (apq == 0.0) { status = ST_STALL; break; }
    p = min(s_rc[0], s_rc[1]);
    q = max(s_rc[0], s_rc[1]);
    // ---- columns p, q: the loads first, the parameters overlap them
    const bool ownp = p >= k0 && p < k0 + nk, ownq = q >= k0 && q < k0 + nk;
    const unsigned pv = version(p), qv = version(q);
    const double* gp = Yc + svd_column_at(pv, p, n, ldc);
    const double* gq = Yc + svd_column_at(qv, q, n, ldc);
    double* newp = Yc + svd_column_at(!pv, p, n, ldc);
    double* newq = Yc + svd_column_at(!qv, q, n, ldc);
    if (lane == svd_version_lane(p)) ver ^= svd_version_bit(p);
    if (lane == svd_version_lane(q)) ver ^= svd_version_bit(q);
    constexpr int kU = 4;
    double t = 0.0, cs = 1.0, sn = 0.0;
    for (int i0 = 0; i0 < m; i0 += kU * NT) {
      double u[kU], w[kU];
#pragma unroll
      for (int e = 0; e < kU; ++e) {
        const int i = min(i0 + e * NT + tid, m - 1);
        u[e] = ld_ag(gp + i);
        w[e] = ld_ag(gq + i);
      }
      if (i0 == 0) rot_params<double>(diag[p], diag[q], apq, t, cs, sn);
#pragma unroll
      for (int e = 0; e < kU; ++e) {
        const int i = i0 + e * NT + tid;
        if (i < m) {
          const double np_ = cs * u[e] + sn * w[e], nq_ = cs * w[e] - sn * u[e];
          colp[i] = np_;
          colq[i] = nq_;
          if (ownp) { Ys[(size_t)(p - k0) * S + i] = np_; }
          if (ownq) { Ys[(size_t)(q - k0) * S + i] = nq_; }
        }
      }
    }
    if (tid == 0 && g == 0 && d.plog && rot < d.logcap) {
      d.plog[2 * rot] = p;
      d.plog[2 * rot + 1] = q;
    }
    ++rot;
    __syncthreads();
    // ---- dot products of this workgroup's columns with p (tasks 0 .. nk - 1) and q, and of p
    // and q with themselves; the last wave rotates this workgroup's part of V^T and stores the
    // columns that it owns
    for (int task = tid; task < 2 * nk + 2; task += NT) {
      const bool self = task >= 2 * nk;
      const bool onp = self ? task == 2 * nk : task < nk;
      const int k = onp ? task : task - nk;
      const double* u = onp ? colp : colq;
      const double x = dot_in_order(u, self ? u : Ys + (size_t)k * S, m);
      if (self) s_new[onp ? 0 : 1] = x;
      else (onp ? xp : xq)[k] = x;
    }
    if (wv == NW - 1) {
      if (d.Vt) {
        for (int i = k0 + lane; i < k0 + nk; i += 64) {
          const double u = d.Vt[(size_t)p * ldv + i], w = d.Vt[(size_t)q * ldv + i];
          d.Vt[(size_t)p * ldv + i] = cs * u + sn * w;
          d.Vt[(size_t)q * ldv + i] = cs * w - sn * u;
        }
      }
      if (ownp)
        for (int i = lane; i < m; i += 64) st_ag(newp + i, colp[i]);
      if (ownq)
        for (int i = lane; i < m; i += 64) st_ag(newq + i, colq[i]);
    }
    __syncthreads();
    // ---- entries of A, row caches (wave 0)
    const double app = s_new[0], aqq = s_new[1];
    if (wv == 0) {
      vp = vq = -1.0;
      ap = aq = 0.0;
      cp = cq = INT_MAX;
      for (int t0 = lane; t0 < nk; t0 += 64) {
        const int k = k0 + t0;
        const double x = xp[t0], y = xq[t0];
        st_ag(d.G + (size_t)p * ldg + k, x);
        st_ag(d.G + (size_t)k * ldg + p, x);
        st_ag(d.G + (size_t)q * ldg + k, y);
        st_ag(d.G + (size_t)k * ldg + q, y);
        const double akk = k == p ? app : (k == q ? aqq : diag[k]);
        const double sp = svd_score<PIV>(akk, app, x);
        const double sq = svd_score<PIV>(akk, aqq, y);
        if (k != p && sp > vp) { vp = sp; cp = k; ap = x; }
        if (k != q && sq > vq) { vq = sq; cq = k; aq = y; }
        if (k == p || k == q) continue;
        double b = best[t0];
        int ak = arg[t0];
        if (ak == p || ak == q) {
          double z = sp, zv = x;
          int col = p;
          if (sq > z) { z = sq; zv = y; col = q; }
          if (z > b || (z == b && col <= ak)) {
            best[t0] = z;
            arg[t0] = col;
            val[t0] = zv;
          } else {
            list[atomicAdd(&s_cnt, 1)] = t0;
          }
        } else {
          double bvv = val[t0];
          if (sp > b || (sp == b && p < ak)) { b = sp; ak = p; bvv = x; }
          if (sq > b || (sq == b && q < ak)) { b = sq; ak = q; bvv = y; }
          best[t0] = b;
          arg[t0] = ak;
          val[t0] = bvv;
        }
      }
    }
    __syncthreads();
    const int cnt = s_cnt;
    if (cnt > 0) {
      // full rescans, one wave per row; the entries stored in this rotation from LDS
      for (int e = wv; e < cnt; e += NW) {
        const int t0 = list[e], k = k0 + t0;
        const double akk = diag[k];
        double bv = -1.0, bav = 0.0;
        int bc = INT_MAX;
        for (int l = lane; l < n; l += 64) {
          if (l == k) continue;
          const double gv = ld_ag(d.G + (size_t)k * ldg + l);
          const double all = l == p ? app : (l == q ? aqq : diag[l]);
          const double z = l == p ? xp[t0] : (l == q ? xq[t0] : gv);
          const double x = svd_score<PIV>(akk, all, z);
          if (x > bv) { bv = x; bc = l; bav = z; }
        }
        const SvdBest r = wave_svd_best(bv, bc, bav);
        if (lane == 0) { best[t0] = r.v; arg[t0] = r.c; val[t0] = r.a; }
      }
      resc += cnt;
      __syncthreads();
    }
    if (tid == 0) {
      s_cnt = 0;
      diag[p] = app;
      diag[q] = aqq;
    }
  }
  if (failed) return;  // the host reports a device error
  __syncthreads();
  for (int k = 0; k < nk; ++k)
    for (int i = tid; i < m; i += NT) d.Y[(size_t)i * d.ldy + k0 + k] = Ys[(size_t)k * S + i];
  if (tid == 0 && resc)
    atomicAdd(reinterpret_cast<unsigned long long*>(&d.ctl->rescans), (unsigned long long)resc);
  if (tid == 0 && g == 0) {
    d.ctl->rotations = rot;
    d.ctl->status = status;
    d.ctl->done = 1;
    d.ctl->final_sel = vsel;
  }
}

// ------------------------------------------------------------------ output
// rank[k] = position of column k in descending order of sigma_k = sqrt(a_kk) (stable);
// S[rank[k]] = sigma_k.
__global__ __launch_bounds__(256) void k_svd_rank(const double* __restrict__ G, int ldg, int n,
                                                  int* __restrict__ rank, double* __restrict__ S) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  const double sk = sqrt(G[(size_t)k * ldg + k]);
  int rk = 0;
  for (int j = 0; j < n; ++j) {
    const double sj = sqrt(G[(size_t)j * ldg + j]);
    rk += (sj > sk) || (sj == sk && j < k);
  }
  rank[k] = rk;
  S[rk] = sk;
}

// U[:, rank k] = b_k / sigma_k (0 when sigma_k == 0); V[:, rank k] = row k of Vt.
__global__ __launch_bounds__(256) void k_svd_vectors(const double* __restrict__ Y, int ldy, int m,
                                                     const double* __restrict__ G, int ldg,
                                                     const double* __restrict__ Vt, int ldvt,
                                                     int n, const int* __restrict__ rank,
                                                     double* __restrict__ U, int ldu,
                                                     double* __restrict__ V, int ldv) {
  const int k = blockIdx.y;
  const int rk = rank[k];
  const double sk = sqrt(G[(size_t)k * ldg + k]);
  for (int i = blockIdx.x * 256 + threadIdx.x; i < m; i += gridDim.x * 256) {
    if (U) U[(size_t)rk * ldu + i] = sk > 0.0 ? Y[(size_t)i * ldy + k] / sk : 0.0;
    if (V && i < n) V[(size_t)rk * ldv + i] = Vt[(size_t)k * ldvt + i];
  }
}

// ------------------------------------------------------------------ launchers
hipError_t launch_svd_load(const double* B, int m, int n, int ldb, double* Y, int ldy, int* flag,
                           hipStream_t s) {
  dim3 g((m + 31) / 32, (n + 31) / 32);
  hipLaunchKernelGGL(k_svd_load, g, dim3(256), 0, s, B, m, n, ldb, Y, ldy, flag);
  return hipGetLastError();
}

hipError_t launch_svd_gram(const double* Y, int ldy, int m, int n, double* G, int ldg,
                           hipStream_t s) {
  dim3 g((n + 15) / 16, (n + 15) / 16);
  hipLaunchKernelGGL(k_svd_gram, g, dim3(256), 0, s, Y, ldy, m, n, G, ldg);
  return hipGetLastError();
}

hipError_t launch_svd_rowmix(const double* Y, int ldy, const double* Q, int ldq, int m, int n,
                             double* Z, int ldz, hipStream_t s) {
  dim3 g((n + 255) / 256, m);
  hipLaunchKernelGGL(k_svd_rowmix, g, dim3(256), 0, s, Y, ldy, Q, ldq, m, n, Z, ldz);
  return hipGetLastError();
}

hipError_t launch_svd_transpose(const double* Q, int ldq, int n, double* Vt, int ldv,
                                hipStream_t s) {
  dim3 g((n + 255) / 256, n);
  hipLaunchKernelGGL(k_svd_transpose, g, dim3(256), 0, s, Q, ldq, n, Vt, ldv);
  return hipGetLastError();
}

static int svd_max_lds() {
  static int v = -1;
  if (v < 0) {
    int dev = 0, x = 65536;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&x, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
      x = 65536;
    v = x;
  }
  return v;
}

bool svd_resident(int m, int n) {
  // two lanes per column; the static LDS of the kernel (1 KB) and a margin stay free
  return n <= kSvdResMaxN && svd_lds_bytes(m, n) + 2048 <= (size_t)svd_max_lds();
}

template <typename K>
static hipError_t svd_launch_main(K fn, int nt, size_t sh, const SDesc& d, hipStream_t s) {
  if (sh > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)fn,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3(1), dim3(nt), sh, s, d);
  return hipGetLastError();
}

template <int PIV>
static hipError_t svd_jacobi_t(const SDesc& d, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_rowbest<PIV>, dim3((d.n + 3) / 4), dim3(256), 0, s, d.G, d.ldg,
                     d.n, d.best, d.arg, d.diag);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (svd_resident(d.m, d.n)) {
    const size_t sh = svd_lds_bytes(d.m, d.n);
    if (d.n <= kSvdResKeepN) return svd_launch_main(k_svd_res<PIV, true>, 256, sh, d, s);
    e = svd_launch_main(k_svd_res<PIV, false>, 256, sh, d, s);
    // A's entries once more, for the final off-norm and the singular values
    return e != hipSuccess ? e : launch_svd_gram(d.Y, d.ldy, d.m, d.n, d.G, d.ldg, s);
  }
  // one workgroup; more lanes once the dot products of a rotation outnumber 256
  if (d.n > 256) return svd_launch_main(k_svd1<PIV, 1024>, 1024, (size_t)d.n * 4, d, s);
  return svd_launch_main(k_svd1<PIV, 256>, 256, (size_t)d.n * 4, d, s);
}

hipError_t launch_svd_jacobi(const SDesc& d, hipStream_t s) {
  if (d.n > kSvdMaxN) return hipErrorInvalidValue;
  if (d.pivot == 0) return svd_jacobi_t<0>(d, s);
  if (d.pivot == 1) return svd_jacobi_t<1>(d, s);
  return svd_jacobi_t<2>(d, s);
}

// Columns per workgroup and workgroups of the several-workgroup kernel; false where a slice
// of B does not fit in LDS (the one-workgroup kernel then reads B from device memory) or the
// one-workgroup resident kernel holds all of it.
static bool svd_mw_shape(int m, int n, int* c, int* G) {
  if (n < 2 || svd_resident(m, n)) return false;
  // four columns at least; all of n <= 3, for the m at which one LDS holds them without the row
  // caches of the resident kernel (4000 x 3: 0.74 ms a call, from device memory 1.2)
  *c = std::min(n, std::max(4, (n + kSvdMwGroups - 1) / kSvdMwGroups));
  *G = (n + *c - 1) / *c;
  return n <= kSvdVersionCols && svd_mw_lds(m, n, *c) + 1024 <= (size_t)svd_max_lds();
}

static inline int svd_mw_ldc(int m) { return (m + 1) & ~1; }

size_t svd_mw_bytes(int m, int n) {
  int c, G;
  if (!svd_mw_shape(m, n, &c, &G)) return 0;
  return sizeof(MwCtl) + ((size_t)2 * G * kSvdMwWords + svd_column_doubles(n, svd_mw_ldc(m))) * 8;
}

int svd_mw_groups(int m, int n) {
  int c, G;
  return svd_mw_shape(m, n, &c, &G) ? G : 0;
}

template <int PIV>
static hipError_t svd_mw_t(const SDesc& d, MwCtl* mc, int c, int G, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_rowbest<PIV>, dim3((d.n + 3) / 4), dim3(256), 0, s, d.G, d.ldg,
                     d.n, d.best, d.arg, d.diag);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  double* xb = (double*)(mc + 1);
  double* Yc = xb + (size_t)2 * G * kSvdMwWords;
  const int ldc = svd_mw_ldc(d.m);
  // Yc[k][i] = Y[i][k], the first copies
  hipLaunchKernelGGL(k_svd_columns, dim3((d.m + 31) / 32, (d.n + 31) / 32), dim3(256), 0, s, d.Y,
                     d.ldy, d.m, d.n, Yc, ldc);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t sh = svd_mw_lds(d.m, d.n, c);
  auto fn = k_svd_mw<PIV>;
  if (sh > 65536) {
    e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3(G * kMwStride), dim3(kSvdMwThreads), sh, s, d, mc, xb, Yc, ldc, G,
                     c);
  return hipGetLastError();
}

hipError_t launch_svd_mw(const SDesc& d, void* buf, hipStream_t s) {
  int c, G;
  if (d.n > kSvdMaxN || !svd_mw_shape(d.m, d.n, &c, &G)) return hipErrorInvalidValue;
  MwCtl* mc = (MwCtl*)buf;
  hipError_t e = launch_zero_words(mc, (int)(sizeof(MwCtl) / 4), s);
  if (e != hipSuccess) return e;
  if (d.pivot == 0) return svd_mw_t<0>(d, mc, c, G, s);
  if (d.pivot == 1) return svd_mw_t<1>(d, mc, c, G, s);
  return svd_mw_t<2>(d, mc, c, G, s);
}

hipError_t launch_svd_out(const double* Y, int ldy, int m, const double* G, int ldg,
                          const double* Vt, int ldvt, int n, int* rank, double* S, double* U,
                          int ldu, double* V, int ldv, hipStream_t s) {
  hipLaunchKernelGGL(k_svd_rank, dim3((n + 255) / 256), dim3(256), 0, s, G, ldg, n, rank, S);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || (!U && !V)) return e;
  dim3 g((m + 255) / 256, n);
  hipLaunchKernelGGL(k_svd_vectors, g, dim3(256), 0, s, Y, ldy, m, G, ldg, Vt, ldvt, n, rank, U,
                     ldu, V, ldv);
  return hipGetLastError();
}

}  // namespace je
