// Eigenpairs of a real symmetric tridiagonal matrix by Cuppen's divide and
// conquer (stage 2 of the dense eigensolve, Sec. 3.2), with the rank-one
// merge solved through the secular equation and Gu-Eisenstat's recomputed
// z vector for orthogonal eigenvectors.
//
// Tree: L = 2^h leaves, leaf boundaries b(i) = floor(i n / L), each leaf at
// most DC_LEAF rows.  Tearing at a boundary k subtracts |e_{k-1}| from
// d_{k-1} and d_k, so T = diag(T1, T2) + rho u u^T with u = (.., 1 | s, ..),
// s = sign(e_{k-1}), rho = |e_{k-1}|.
//
// Merge of (lam1, Q1) and (lam2, Q2) (m = n1 + n2 rows):
//   z = (last row of Q1, s * first row of Q2) / sqrt 2, rho' = 2 rho,
//   D + rho' z z^T with D = diag(lam1, lam2) sorted (parallel merge by binary
//   search); deflation (sequential scan): |rho' z_j| <= tol, or a Givens
//   rotation of a close pair (d_p, d_j) with |(d_j - d_p) c s| <= tol;
//   secular equation f(x) = 1 + rho' sum z_i^2/(d_i - x) = 0 for the K
//   remaining roots (one wavefront per root, origin shifted to the nearer
//   pole, rational two-pole interpolation safeguarded by bisection);
//   zhat_i^2 = prod_j (x_j - d_i) / (rho' prod_{j != i} (d_j - d_i));
//   u_ij = zhat_i / (d_i - x_j) normalised; new vectors = Q_nd U (FP64 MFMA
//   GEMM); eigenvalues merged in ascending order (rank by counting).
// All per-merge scratch lives at the merge's own index range [s, t) of n-long
// arrays, so every merge of a tree level runs in the same launches.
//
// Grouped execution: the kernels read each problem's tree and buffers from a
// device table (DcProb); the grid's z dimension enumerates the problems and y
// the merges (the deflation scan's x both), so one launch serves a tree level of
// every matrix of a batch.  A single tridiagonal problem is the one-entry case.
#include <float.h>
#include <vector>
#include "common.h"
#include "stages.h"
#include "gemm_core.h"
#include "table.h"

namespace mmf {

constexpr int DC_LEAF = 16;
constexpr int DC_CNT = 5;     // per merge: K, rotations, deflated, top-only, top-only + mixed columns
constexpr double DC_EPS = DBL_EPSILON;

struct DcWs {
  double *dw, *lam, *T1, *T2;
  double *es, *scl;           // scaled off-diagonal; the power of two, its reciprocal, nonzero once an eigenvalue is NaN
  double *ds, *zs, *dn, *zn, *ddef, *rc, *rs, *lamt, *zhat, *rho;
  int32_t *src, *ndidx, *dfidx, *rp, *rj, *lamo, *colmap, *cnt;   // cnt: [DC_CNT * n] per merge
  int32_t *ctype, *perm;      // child type of each column (1 top, 2 bottom, 3 both); T1/T2 slot of each kept column
  size_t bytes;
};

inline DcWs stedc_ws(int64_t n, void *base) {
  Carver cv(base);
  DcWs w;
  const size_t N = (size_t)(n > 0 ? n : 1);
  w.dw = cv.take<double>(N);
  w.lam = cv.take<double>(N);
  w.es = cv.take<double>(N);
  w.scl = cv.take<double>(3);
  w.T1 = cv.take<double>(N * N);
  w.T2 = cv.take<double>(N * N);
  w.ds = cv.take<double>(N);
  w.zs = cv.take<double>(N);
  w.dn = cv.take<double>(N);
  w.zn = cv.take<double>(N);
  w.ddef = cv.take<double>(N);
  w.rc = cv.take<double>(N);
  w.rs = cv.take<double>(N);
  w.lamt = cv.take<double>(N);
  w.zhat = cv.take<double>(N);
  w.rho = cv.take<double>(N);
  w.src = cv.take<int32_t>(N);
  w.ndidx = cv.take<int32_t>(N);
  w.dfidx = cv.take<int32_t>(N);
  w.rp = cv.take<int32_t>(N);
  w.rj = cv.take<int32_t>(N);
  w.lamo = cv.take<int32_t>(N);
  w.colmap = cv.take<int32_t>(N);
  w.cnt = cv.take<int32_t>(DC_CNT * N);
  w.ctype = cv.take<int32_t>(N);
  w.perm = cv.take<int32_t>(N);
  w.bytes = cv.used();
  return w;
}

size_t stedc_ws_bytes(int64_t n) { return stedc_ws(n, nullptr).bytes + 512; }

struct DcProb {
  int64_t n, ldz, L;
  int32_t h;
  int32_t sec_max, leaf_max;     // iteration caps: secular steps per root, QL steps per eigenvalue
  int32_t window;                // eigenvectors wanted: all (0), or those of eigenvalues in [vl, vu)
  double vl, vu;
  double *d;
  const double *e0;              // caller's off-diagonal; the kernels use e = w.es
  const double *e;
  double *Z;
  int32_t *info;
  DcWs w;
};

inline int dc_depth(int64_t n) {
  int h = 0;
  while (((n + ((int64_t)1 << h) - 1) >> h) > DC_LEAF) ++h;
  return h;
}

__device__ __host__ inline int64_t dc_b(int64_t i, int64_t n, int64_t L) { return (i * n) / L; }

struct MergeGeom {
  int64_t s, mid, t, m, n1;
};
__device__ inline MergeGeom dc_geom(int64_t n, int64_t L, int lev, int64_t g) {
  MergeGeom q;
  const int64_t span = (int64_t)1 << lev;
  q.s = dc_b(g * span, n, L);
  q.mid = dc_b(g * span + span / 2, n, L);
  q.t = dc_b((g + 1) * span, n, L);
  q.m = q.t - q.s;
  q.n1 = q.mid - q.s;
  return q;
}

// ------------------------------------------------------------------ tearing
// True when x is one of the leaf boundaries b(j) = floor(j n / L), 0 < j < L.
__device__ inline bool dc_is_boundary(int64_t x, int64_t n, int64_t L) {
  if (x <= 0 || x >= n) return false;
  const int64_t j = (x * L + n - 1) / n;          // smallest j with j n / L >= x
  return j >= 1 && j < L && dc_b(j, n, L) == x;
}

// Status word cleared and the power of two that brings the largest entry to
// [1/2, 1): the merges form squares and reciprocals of differences, which a
// matrix of norm 1e-150 or 1e150 would push out of range.  Exact, so that any
// other matrix gives the same bits with and without it.
__global__ void __launch_bounds__(1024) dc_scale(const DcProb *pr) {
  __shared__ double sh[16];
  const DcProb &q = pr[blockIdx.z];
  const int64_t n = q.n;
  double m = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 1024) {
    m = fmax(m, fabs(q.d[i]));
    if (i < n - 1) m = fmax(m, fabs(q.e0[i]));
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int g = 1; g < 16; ++g) m = fmax(m, sh[g]);
  int ex = 0;
  if (m > 0.0 && m <= DBL_MAX) (void)frexp(m, &ex);
  ex = ex > 1000 ? 1000 : (ex < -1000 ? -1000 : ex);
  q.w.scl[0] = ldexp(1.0, -ex);
  q.w.scl[1] = ldexp(1.0, ex);
  q.w.scl[2] = 0.0;
  *q.info = 0;
}

// Eigenvalues are ranked by comparisons, and the ranks become positions in
// arrays and columns of Z: a NaN (which a NaN or infinite entry of the matrix
// spreads) would leave positions unset that are then used as indices.  It counts
// as zero in every ranking; the call reports no convergence and returns NaN.
__device__ inline void dc_not_a_number(const DcProb &P) {
  P.w.scl[2] = 1.0;
  *P.info = MMF_ERR_NO_CONVERGENCE;
}

// es = e and dw = d scaled, with |e_{k-1}| taken from d_{k-1} and d_k at every
// boundary k (one thread per row; boundaries are at least one leaf apart).
__global__ void dc_tear(const DcProb *pr) {
  const DcProb &q = pr[blockIdx.z];
  const int64_t n = q.n, L = q.L;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double sc = q.w.scl[0];
  double v = q.d[i] * sc;
  if (dc_is_boundary(i + 1, n, L)) v -= fabs(q.e0[i] * sc);       // i = k - 1
  if (dc_is_boundary(i, n, L)) v -= fabs(q.e0[i - 1] * sc);       // i = k
  q.w.dw[i] = v;
  if (i < n - 1) q.w.es[i] = q.e0[i] * sc;
}

// ------------------------------------------------------------------ leaves
// One wavefront per leaf: implicit QL with Wilkinson shifts (the textbook
// symmetric tridiagonal QL iteration: Bowdler, Martin, Reinsch and Wilkinson,
// Numer. Math. 11 (1968), the tql2 procedure; Golub and Van Loan, Sec. 8.3).
// Lane i holds d_i and e_i; every lane runs the scalar recurrence (identical
// values, d_i and e_i fetched by lane reads) and rotates its own row of Z.
// The rotations are one chain of about 1.3 m^2 steps, so a step's latency and
// the leaf size are what counts.  With d and e in LDS behind barriers, hypot
// and two divisions a step, leaves of up to 64 took 797 us at order 82 and
// 1430 at 1715; this form 419 and 728.  Whole solves with leaves of 64 / 32 /
// 16 (each halving adds a merge level, about 0.1 ms at small orders): order 82
// 1.35 / 1.14 / 1.13 ms, dressed qubit (450) 7.06 / 6.62 / 6.51 ms, order 1715
// 26.7 / 26.3 / 26.2 ms, band window 12816 259 ms each.
__global__ void __launch_bounds__(64) dc_leaf(const DcProb *pr) {
  __shared__ double Zl[DC_LEAF * 64];               // column c, row r at 64 c + r
  __shared__ int perm[DC_LEAF];
  const DcProb &q = pr[blockIdx.z];
  const int64_t n = q.n, L = q.L, ldz = q.ldz;
  if ((int64_t)blockIdx.x >= L || n <= 0) return;
  const double *dw = q.w.dw, *e = q.e;
  double *Z = q.Z, *lam = q.w.lam;
  const int64_t s = dc_b(blockIdx.x, n, L);
  const int m = (int)(dc_b(blockIdx.x + 1, n, L) - s);
  const int r = threadIdx.x;
  double dd = r < m ? dw[s + r] : 0.0;
  double ee = r < m - 1 ? e[s + r] : 0.0;
  for (int c = 0; c < m; ++c) Zl[c * 64 + r] = (c == r) ? 1.0 : 0.0;
  __syncthreads();
  bool fail = false;
  for (int l = 0; l < m; ++l) {
    int iter = 0;
    while (true) {
      // first negligible e from l on (e_{m-1} = 0)
      const bool neg = fabs(ee) <= DC_EPS * (fabs(dd) + fabs(__shfl_down(dd, 1, 64)));
      const uint64_t mask = __ballot(neg && r < m - 1) >> l;
      const int mm = mask ? l + __builtin_ctzll(mask) : m - 1;
      if (mm == l) break;
      if (++iter > q.leaf_max) { fail = true; break; }
      const double dl = lane_get(dd, l), el = lane_get(ee, l);
      double g = (lane_get(dd, l + 1) - dl) / (2.0 * el);
      double rr = hypot(g, 1.0);
      g = lane_get(dd, mm) - dl + el / (g + copysign(rr, g));
      double sn = 1.0, c = 1.0, p = 0.0;
      double zc = Zl[mm * 64 + r];                  // column i + 1 of this row
      int i = mm - 1;
      bool restart = false;
      for (; i >= l; --i) {
        const double ei = lane_get(ee, i), di = lane_get(dd, i), di1 = lane_get(dd, i + 1);
        const double zi = Zl[i * 64 + r];
        const double f = sn * ei;
        const double b = c * ei;
        const double h = fma(f, f, g * g);
        if (h > 1e-280 && h < 1e280) {              // uniform
          const double ri = rsqrt(h);
          rr = h * ri;
          sn = f * ri;
          c = g * ri;
        } else {
          rr = hypot(f, g);
          if (rr == 0.0) {
            if (r == i + 1) { dd -= p; ee = 0.0; }
            if (r == mm) ee = 0.0;
            restart = true;
            break;
          }
          sn = f / rr;
          c = g / rr;
        }
        if (r == i + 1) ee = rr;
        g = di1 - p;
        rr = (di - g) * sn + 2.0 * c * b;
        p = sn * rr;
        if (r == i + 1) dd = g + p;
        g = c * rr - b;
        Zl[(i + 1) * 64 + r] = sn * zi + c * zc;
        zc = c * zi - sn * zc;
      }
      Zl[(i + 1) * 64 + r] = zc;
      if (restart) continue;
      if (r == l) { dd -= p; ee = g; }
      if (r == mm) ee = 0.0;
    }
    if (fail) break;
  }
  if (fail && r == 0) *q.info = MMF_ERR_NO_CONVERGENCE;
  if (dd != dd) {
    dc_not_a_number(q);
    dd = 0.0;
  }
  // ascending order (selection by rank; ties by index)
  int rank = 0;
  for (int j = 0; j < m; ++j) {
    const double u = lane_get(dd, j);
    rank += (u < dd) || (u == dd && j < r);
  }
  if (r < m) {
    perm[rank] = r;
    lam[s + rank] = dd;
  }
  __syncthreads();
  if (r < m)
    for (int c = 0; c < m; ++c) Z[(s + r) + (s + c) * ldz] = Zl[perm[c] * 64 + r];
}

// ------------------------------------------------------------------ merge: prepare
__device__ void dc_sort(const DcProb &P, int lev, int64_t bx) {
  const int64_t n = P.n, L = P.L, ldz = P.ldz;
  const double *e = P.e, *lam = P.w.lam, *Z = P.Z;
  double *ds = P.w.ds, *zs = P.w.zs, *rho = P.w.rho;
  int32_t *src = P.w.src;
  const MergeGeom q = dc_geom(n, L, lev, blockIdx.y);
  const int64_t j = bx * blockDim.x + threadIdx.x;
  if (j >= q.m) return;
  const double ek = e[q.mid - 1];
  const double sg = ek >= 0.0 ? 1.0 : -1.0;
  const double inv_sqrt2 = 0.70710678118654752440;
  double dv, zv;
  int64_t pos;
  const double *L2 = lam + q.mid;
  const int64_t n2 = q.t - q.mid;
  if (j < q.n1) {
    dv = lam[q.s + j];
    zv = Z[(q.mid - 1) + (q.s + j) * ldz];
    int64_t lo = 0, hi = n2;           // count of right values < dv
    while (lo < hi) { const int64_t md = (lo + hi) >> 1; if (L2[md] < dv) lo = md + 1; else hi = md; }
    pos = j + lo;
  } else {
    const int64_t jj = j - q.n1;
    dv = lam[q.mid + jj];
    zv = sg * Z[q.mid + (q.mid + jj) * ldz];
    const double *L1 = lam + q.s;
    int64_t lo = 0, hi = q.n1;         // count of left values <= dv
    while (lo < hi) { const int64_t md = (lo + hi) >> 1; if (L1[md] <= dv) lo = md + 1; else hi = md; }
    pos = jj + lo;
  }
  ds[q.s + pos] = dv;
  zs[q.s + pos] = zv * inv_sqrt2;
  src[q.s + pos] = (int32_t)j;
  P.w.ctype[q.s + pos] = j < q.n1 ? 1 : 2;    // child whose rows the column spans
  if (j == 0) rho[q.s] = 2.0 * fabs(ek);
}

// Off-diagonal blocks of the merged block start as exact zeros: row block rb,
// chunk ch of 64 columns.
__device__ void dc_zero_off(const DcProb &P, int lev, int64_t rb, int64_t ch) {
  const MergeGeom q = dc_geom(P.n, P.L, lev, blockIdx.y);
  const int64_t r = rb * blockDim.x + threadIdx.x;
  if (r >= q.m) return;
  const bool rl = r < q.n1;
  const int64_t c0 = ch * 64;
  const int64_t c1 = (c0 + 64 < q.m) ? c0 + 64 : q.m;
  for (int64_t c = c0; c < c1; ++c) {
    const bool cl = c < q.n1;
    if (rl != cl) P.Z[(q.s + r) + (q.s + c) * P.ldz] = 0.0;
  }
}

// The two together: nrow blocks of the sorted union, then the zero blocks.
// (Steps of a merge that do not need one another share a launch: seven launches
// a level instead of eleven, each as long as its longer step: whole solves
// 0.675 -> 0.619 ms at order 82, 5.04 -> 4.88 at 450, 21.9 -> 21.6 at 1715.)
__global__ void __launch_bounds__(256) dc_prep(const DcProb *pr, int lev, int nrow) {
  const DcProb &P = pr[blockIdx.z];
  if (lev > P.h || (int64_t)blockIdx.y >= (P.L >> lev)) return;
  const int64_t x = (int64_t)blockIdx.x - nrow;
  if (x < 0) dc_sort(P, lev, blockIdx.x);
  else dc_zero_off(P, lev, x % nrow, x / nrow);
}

// ------------------------------------------------------------------ merge: deflation scan
// One wavefront per merge.  The scan is sequential only where it rotates:
// each test involves the last kept entry, which a rotation changes.  Chunks of
// 64 entries are read at once (one per lane, the next chunk ahead); if no
// kept entry of a chunk forms a close pair with the kept entry before it, the
// whole chunk is taken in parallel (slots by ballots), otherwise entry by
// entry with lane broadcasts.  The current last kept entry (its z, d and child
// type) stays in registers.  Each kept column's child type is final when it is
// kept (only the later entry of a rotated pair changes type), so the slots of
// the kept columns grouped [top only | both | bottom only] are then formed in
// parallel, 64 at a time.  Entry by entry throughout took 995 us a level at
// order 12816 (85 at 450), this form 47.
__global__ void __launch_bounds__(64) dc_deflate(const DcProb *pr, int lev, int64_t Gmax) {
  const DcProb &P = pr[blockIdx.x / Gmax];
  const int64_t g = blockIdx.x % Gmax;
  if (lev > P.h || g >= (P.L >> lev)) return;
  double *ds = P.w.ds, *zs = P.w.zs, *rc = P.w.rc, *rs = P.w.rs;
  const double *rho = P.w.rho;
  int32_t *ndidx = P.w.ndidx, *dfidx = P.w.dfidx, *rp = P.w.rp, *rj = P.w.rj, *cnt = P.w.cnt;
  int32_t *ctype = P.w.ctype, *perm = P.w.perm;
  const MergeGeom q = dc_geom(P.n, P.L, lev, g);
  const int64_t s = q.s, m = q.m;
  const int lane = threadIdx.x;
  const bool w0 = lane == 0;
  const uint64_t below = (1ull << lane) - 1;
  const double rh = rho[s];
  double dmax = fmax(fabs(ds[s]), fabs(ds[s + m - 1]));
  const double tol = 8.0 * DC_EPS * fmax(dmax, rh);
  int32_t K = 0, ND = 0, R = 0, c1 = 0, c3 = 0;
  int64_t prev = -1;
  double zp = 0.0, dp = 0.0;                       // z, d of the last kept entry
  int32_t tp = 0;                                  // its child type
  // close pair (a Givens rotation of z_a, z_b leaves |(d_b - d_a) c s| <= tol):
  // z of a kept entry is at least 8 eps, so the products cannot underflow
  auto close = [&](double za, double da, double zb, double db) {
    return fabs((db - da) * za * zb) <= tol * fma(za, za, zb * zb);
  };
  double zn = lane < m ? zs[s + lane] : 0.0, dn = lane < m ? ds[s + lane] : 0.0;
  int32_t tn = lane < m ? ctype[s + lane] : 0;
  for (int64_t j0 = 0; j0 < m; j0 += 64) {
    const double zl = zn, dl = dn;
    const int32_t tl = tn;
    const int nu = (int)((m - j0 < 64) ? m - j0 : 64);
    {
      const int64_t jn = j0 + 64 + lane;
      zn = jn < m ? zs[s + jn] : 0.0;
      dn = jn < m ? ds[s + jn] : 0.0;
      tn = jn < m ? ctype[s + jn] : 0;
    }
    const bool kept = lane < nu && !(rh * fabs(zl) <= tol);
    const uint64_t mk = __ballot(kept), md = __ballot(lane < nu && !kept);
    const uint64_t before = mk & below;
    const int pl = before ? 63 - __builtin_clzll(before) : 0;
    const double zq = __shfl(zl, pl, 64), dq = __shfl(dl, pl, 64);
    const int32_t tq = __shfl(tl, pl, 64);
    const double zb = before ? zq : zp, db = before ? dq : dp;
    const int32_t tb = before ? tq : tp;
    const bool has = kept && (before || prev >= 0);
    if (__ballot(has && close(zb, db, zl, dl)) == 0) {
      if (lane < nu && !kept) dfidx[s + ND + __popcll(md & below)] = (int32_t)(j0 + lane);
      ND += __popcll(md);
      if (mk) {
        // every kept entry settles the kept entry before it
        const int32_t base = prev >= 0 ? K : K - 1;
        if (has) {
          const int32_t pos = base + __popcll(before);
          ndidx[s + pos] = (int32_t)(before ? j0 + pl : prev);
          perm[s + pos] = tb;                      // child type for now, slot below
        }
        c1 += __popcll(__ballot(has && tb == 1));
        c3 += __popcll(__ballot(has && tb == 3));
        K = base + __popcll(mk);
        const int last = 63 - __builtin_clzll(mk);
        prev = j0 + last;
        zp = lane_get(zl, last);
        dp = lane_get(dl, last);
        tp = __builtin_amdgcn_readlane(tl, last);
      }
      continue;
    }
    for (int u = 0; u < nu; ++u) {
      const int64_t j = j0 + u;
      const double zj = lane_get(zl, u);
      if (rh * fabs(zj) <= tol) {
        if (w0) dfidx[s + ND] = (int32_t)j;
        ++ND;
        continue;
      }
      const double dj = lane_get(dl, u);
      const int32_t tj = __builtin_amdgcn_readlane(tl, u);
      if (prev < 0) {
        prev = j; zp = zj; dp = dj; tp = tj;
        continue;
      }
      if (close(zp, dp, zj, dj)) {
        const double tt = hypot(zj, zp);
        const double cv = zj / tt, sv = zp / tt;
        const double dpn = cv * cv * dp + sv * sv * dj, djn = sv * sv * dp + cv * cv * dj;
        if (w0) {
          zs[s + j] = tt;
          zs[s + prev] = 0.0;
          ds[s + prev] = dpn;
          ds[s + j] = djn;
          rp[s + R] = (int32_t)prev;
          rj[s + R] = (int32_t)j;
          rc[s + R] = cv;
          rs[s + R] = sv;
          ctype[s + j] = tj | tp;                  // the kept column now spans both children's rows
          dfidx[s + ND] = (int32_t)prev;
        }
        ++R;
        ++ND;
        prev = j; zp = tt; dp = djn; tp = tj | tp;
      } else {
        if (w0) {
          ndidx[s + K] = (int32_t)prev;
          perm[s + K] = tp;                        // child type for now, slot below
        }
        ++K;
        c1 += tp == 1;
        c3 += tp == 3;
        prev = j; zp = zj; dp = dj; tp = tj;
      }
    }
  }
  if (prev >= 0) {
    if (w0) {
      ndidx[s + K] = (int32_t)prev;
      perm[s + K] = tp;
    }
    ++K;
    c1 += tp == 1;
    c3 += tp == 3;
  }
  // kept columns grouped [top only | both | bottom only] (d order inside each
  // group): the merge GEMM then multiplies the top rows by the first two
  // groups and the bottom rows by the last two only
  __threadfence();
  int32_t p1 = 0, p3 = c1, p2 = c1 + c3;
  for (int32_t k0 = 0; k0 < K; k0 += 64) {
    const int32_t k = k0 + lane;
    const int32_t t = k < K ? perm[s + k] : 0;
    const uint64_t b1 = __ballot(t == 1), b3 = __ballot(t == 3), b2 = __ballot(k < K && t != 1 && t != 3);
    if (k < K) {
      const int32_t pos = t == 1 ? p1 + __popcll(b1 & below)
                                 : (t == 3 ? p3 + __popcll(b3 & below) : p2 + __popcll(b2 & below));
      perm[s + k] = pos;
    }
    p1 += __popcll(b1);
    p3 += __popcll(b3);
    p2 += __popcll(b2);
  }
  if (w0) {
    cnt[DC_CNT * g + 0] = K;
    cnt[DC_CNT * g + 1] = R;
    cnt[DC_CNT * g + 2] = ND;
    cnt[DC_CNT * g + 3] = c1;
    cnt[DC_CNT * g + 4] = c1 + c3;
  }
}

// ------------------------------------------------------------------ merge: rotate + gather
// Thread = row of the merged block: applies the deflation rotations in order
// to its row of Z (a row's rotations chain through shared columns).
__global__ void dc_rotate(const DcProb *pr, int lev) {
  const DcProb &P = pr[blockIdx.z];
  const int64_t g = blockIdx.y;
  if (lev > P.h || g >= (P.L >> lev)) return;
  const int64_t ldz = P.ldz;
  const int32_t *src = P.w.src, *ndidx = P.w.ndidx, *dfidx = P.w.dfidx, *rp = P.w.rp, *rj = P.w.rj;
  const int32_t *cnt = P.w.cnt;
  const double *rc = P.w.rc, *rs = P.w.rs, *ds = P.w.ds, *zs = P.w.zs;
  double *dn = P.w.dn, *zn = P.w.zn, *ddef = P.w.ddef;
  const MergeGeom q = dc_geom(P.n, P.L, lev, g);
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= q.m) return;
  const int64_t s = q.s;
  const int32_t K = cnt[DC_CNT * g], R = cnt[DC_CNT * g + 1], ND = cnt[DC_CNT * g + 2];
  double *zrow = P.Z + (s + r);
  for (int32_t k = 0; k < R; ++k) {
    const int64_t cp = s + src[s + rp[s + k]], cj = s + src[s + rj[s + k]];
    const double c = rc[s + k], sn = rs[s + k];
    const double zp = zrow[cp * ldz], zj = zrow[cj * ldz];
    zrow[cp * ldz] = c * zp - sn * zj;
    zrow[cj * ldz] = sn * zp + c * zj;
  }
  if (r < K) {
    dn[s + r] = ds[s + ndidx[s + r]];
    zn[s + r] = zs[s + ndidx[s + r]];
  }
  if (r < ND) ddef[s + r] = ds[s + dfidx[s + r]];
}

// Gathers the non-deflated columns (in d order, at their kept-column slots)
// into T1[:, 0:K] and the deflated ones into T1[:, K:m].  Workgroup (row tile
// x, y = merge g * nch + column chunk): a chunk of 64 output columns, their
// column pairs looked up once into LDS (three dependent reads each), thread =
// row.  Chunks of 256 columns with the look-up in the copy loop took 131 us a
// level at order 450 (403 at 12816), this form 19 (154).
constexpr int DC_GCOLS = 64;
__device__ void dc_gather(const DcProb &P, int lev, int64_t rb, int64_t ch) {
  __shared__ int32_t cfrom[DC_GCOLS], cto[DC_GCOLS];
  const int64_t g = blockIdx.y;
  const int64_t n = P.n, ldz = P.ldz;
  const int32_t *src = P.w.src, *ndidx = P.w.ndidx, *dfidx = P.w.dfidx, *perm = P.w.perm;
  const int32_t *cnt = P.w.cnt;
  const MergeGeom q = dc_geom(n, P.L, lev, g);
  const int64_t r0 = rb * blockDim.x, o0 = ch * DC_GCOLS;
  if (r0 >= q.m || o0 >= q.m) return;
  const int64_t s = q.s;
  const int32_t K = cnt[DC_CNT * g];
  const int nc = (int)(q.m - o0 < DC_GCOLS ? q.m - o0 : DC_GCOLS);
  if ((int)threadIdx.x < nc) {
    const int64_t o = o0 + threadIdx.x;
    cfrom[threadIdx.x] = (int32_t)s + (o < K ? src[s + ndidx[s + o]] : src[s + dfidx[s + (o - K)]]);
    cto[threadIdx.x] = (int32_t)s + (o < K ? perm[s + o] : (int32_t)o);
  }
  __syncthreads();
  const int64_t r = r0 + threadIdx.x;
  if (r >= q.m) return;
  const double *zrow = P.Z + (s + r);
  double *trow = P.w.T1 + (s + r);
#pragma unroll 8
  for (int c = 0; c < nc; ++c) trow[cto[c] * n] = zrow[cfrom[c] * ldz];
}

// ------------------------------------------------------------------ merge: secular equation
// One wavefront per root k of f(x) = 1 + rho sum_i z_i^2/(d_i - x): rational
// interpolation with the poles beside the root exact, from the root of the
// two poles and of the rest of f at the middle of the interval.  Where three
// steps did not bring f to a tenth (clustered poles on one side: the model's
// steps only halve the distance) the next one divides the bracket, by orders of
// magnitude: the geometric mean, or a thousandth while one end is the pole.
// Bound: the longest chain of steps of any root.  Starting in the middle and
// halving whenever the bracket had not halved (which it does not where the steps
// come from one side), single roots took 20 to 30 steps where the mean is 5, now
// 7 to 11, at most about 20, with a mean of 3 to 4: 10 us a merge at order 82, 14 at 450, 24 at 1715,
// against 24, 36 and 56.
__device__ void dc_roots(const DcProb &P, int lev) {
  const int64_t g = blockIdx.y;
  const double *dn = P.w.dn, *zn = P.w.zn, *rho = P.w.rho;
  const int32_t *cnt = P.w.cnt;
  int32_t *lamo = P.w.lamo, *info = P.info;
  double *lamt = P.w.lamt;
  const MergeGeom q = dc_geom(P.n, P.L, lev, g);
  const int K = cnt[DC_CNT * g];
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (k >= K) return;
  const int64_t s = q.s;
  const double *d = dn + s, *z = zn + s;
  const double rh = rho[s];
  if (K == 1) {
    if (lane == 0) { lamo[s] = 0; lamt[s] = rh * z[0] * z[0]; }
    return;
  }
  int o;
  double lo, hi, c0 = 0.0;
  if (k < K - 1) {
    const double delta = d[k + 1] - d[k];
    const double mid = 0.5 * delta;
    for (int i = lane; i < K; i += 64) {
      const double t = z[i] * z[i] / ((d[i] - d[k]) - mid);
      c0 += i == k || i == k + 1 ? 0.0 : t;
    }
    c0 = 1.0 + rh * wave_sum(c0);                   // f at the middle without the two poles beside the root
    const double f = c0 + rh * (z[k + 1] * z[k + 1] - z[k] * z[k]) / mid;
    if (f >= 0.0) { o = k; lo = 0.0; hi = mid; }
    else { o = k + 1; lo = -mid; hi = 0.0; }
  } else {
    double zz = 0.0;
    for (int i = lane; i < K; i += 64) zz += z[i] * z[i];
    zz = wave_sum(zz);
    o = K - 1;
    lo = 0.0;
    hi = rh * zz;
  }
  const double dorg = d[o];
  const double pk = d[k] - dorg;                  // left pole (relative)
  const double qk = (k < K - 1) ? d[k + 1] - dorg : 0.0;   // right pole
  // root in (lo, hi) of c + b1 / (pk - x) + b2 / (qk - x), else the middle
  const auto rational = [&](double c, double b1, double b2) {
    const double A = c, B = -(c * (pk + qk) + b1 + b2), Cc = c * pk * qk + b1 * qk + b2 * pk;
    double x1 = NAN, x2 = NAN;
    if (A == 0.0) {
      x1 = -Cc / B;
    } else {
      double disc = B * B - 4.0 * A * Cc;
      if (disc < 0.0) disc = 0.0;
      const double sq = sqrt(disc);
      const double qq = -0.5 * (B + copysign(sq, B));
      x1 = qq / A;
      if (qq != 0.0) x2 = Cc / qq;
    }
    if (x1 > lo && x1 < hi) return x1;
    return x2 > lo && x2 < hi ? x2 : 0.5 * (lo + hi);
  };
  double tau = k < K - 1 ? rational(c0, rh * z[k] * z[k], rh * z[k + 1] * z[k + 1]) : 0.5 * (lo + hi);
  double lastf = INFINITY;
  bool conv = false;
  for (int it = 0; it < P.sec_max; ++it) {
    double ps = 0.0, ph = 0.0, dps = 0.0, dph = 0.0;
    for (int i = lane; i < K; i += 64) {
      const double den = (d[i] - dorg) - tau;
      const double t = z[i] * z[i] / den;
      if (i <= k) { ps += t; dps += t / den; } else { ph += t; dph += t / den; }
    }
    ps = rh * wave_sum(ps);
    ph = rh * wave_sum(ph);
    dps = rh * wave_sum(dps);
    dph = rh * wave_sum(dph);
    const double f = 1.0 + ps + ph;
    if (f < 0.0) lo = tau; else hi = tau;
    // rounding bound of f at tau: eps times the absolute sum of its terms
    // (each of the two partial sums has terms of one sign)
    const double errb = 8.0 * DC_EPS * (1.0 + fabs(ps) + fabs(ph));
    if (fabs(f) <= errb || (hi - lo) <= 4.0 * DC_EPS * fmax(fabs(lo), fabs(hi))) { conv = true; break; }
    const double b1 = dps * (pk - tau) * (pk - tau);
    const double a1 = ps - b1 / (pk - tau);
    double xn;
    if (k < K - 1) {
      const double b2 = dph * (qk - tau) * (qk - tau);
      const double a2 = ph - b2 / (qk - tau);
      xn = rational(1.0 + a1 + a2, b1, b2);
    } else {
      const double c = 1.0 + a1 + ph;
      xn = (c != 0.0) ? pk + b1 / c : 0.5 * (lo + hi);
      if (!(xn > lo && xn < hi)) xn = 0.5 * (lo + hi);
    }
    if (it % 3 == 2) {
      if (fabs(f) > 0.1 * lastf) {
        const double near = fmin(fabs(lo), fabs(hi)), far = fmax(fabs(lo), fabs(hi));   // from the pole d[o]
        const double g = near == 0.0 ? 1e-3 * far : (far > 4.0 * near ? sqrt(near * far) : 0.5 * (near + far));
        xn = hi > 0.0 ? g : -g;
      }
      lastf = fabs(f);
    }
    tau = xn;
  }
  if (lane == 0) {
    lamo[s + k] = o;
    lamt[s + k] = tau;
    if (!conv) *info = MMF_ERR_NO_CONVERGENCE;
  }
}

// nroot workgroups of roots, then the gathered columns (nrow row blocks of each chunk).
__global__ void __launch_bounds__(256) dc_secular(const DcProb *pr, int lev, int nroot, int nrow) {
  const DcProb &P = pr[blockIdx.z];
  if (lev > P.h || (int64_t)blockIdx.y >= (P.L >> lev)) return;
  const int64_t x = (int64_t)blockIdx.x - nroot;
  if (x < 0) dc_roots(P, lev);
  else dc_gather(P, lev, x % nrow, x / nrow);
}

// zhat_i^2 = (x_{K-1} - d_i)/rho * prod_{j<i} (x_j - d_i)/(d_j - d_i)
//                                 * prod_{i<=j<K-1} (x_j - d_i)/(d_{j+1} - d_i)
__device__ void dc_zhat(const DcProb &P, int lev) {
  const int64_t g = blockIdx.y;
  const double *dn = P.w.dn, *zn = P.w.zn, *rho = P.w.rho, *lamt = P.w.lamt;
  const int32_t *cnt = P.w.cnt, *lamo = P.w.lamo;
  double *zhat = P.w.zhat;
  const MergeGeom q = dc_geom(P.n, P.L, lev, g);
  const int K = cnt[DC_CNT * g];
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= K) return;
  const int64_t s = q.s;
  const double *d = dn + s;
  const double di = d[i];
  double prod = 1.0;
  for (int j = lane; j < K - 1; j += 64) {
    const double num = (d[lamo[s + j]] - di) + lamt[s + j];
    const double den = (j < i) ? (d[j] - di) : (d[j + 1] - di);
    prod *= num / den;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) prod *= __shfl_xor(prod, o, 64);
  if (lane == 0) {
    const double last = ((d[lamo[s + K - 1]] - di) + lamt[s + K - 1]) / rho[s];
    const double v = sqrt(fmax(prod * last, 0.0));
    zhat[s + i] = copysign(v, zn[s + i]);
  }
}

// Whether root j of a merge needs its eigenvector: every root below the top
// merge, there those of the wanted window (compared as the caller will see them).
__device__ inline bool dc_wanted(const DcProb &P, int lev, int64_t s, int j) {
  if (lev < P.h || !P.window) return true;
  const double v = (P.w.dn[s + P.w.lamo[s + j]] + P.w.lamt[s + j]) * P.w.scl[1];
  return v >= P.vl && v < P.vu;
}

// Column j of the rank-one eigenvector matrix U (T2 block, ld n).
__global__ void __launch_bounds__(256) dc_vectors(const DcProb *pr, int lev) {
  __shared__ double sh[4];
  const DcProb &P = pr[blockIdx.z];
  const int64_t g = blockIdx.y;
  if (lev > P.h || g >= (P.L >> lev)) return;
  const int64_t n = P.n;
  const double *dn = P.w.dn, *lamt = P.w.lamt, *zhat = P.w.zhat;
  const int32_t *cnt = P.w.cnt, *lamo = P.w.lamo;
  double *T2 = P.w.T2;
  const MergeGeom q = dc_geom(n, P.L, lev, g);
  const int K = cnt[DC_CNT * g];
  const int j = blockIdx.x;
  if (j >= K || !dc_wanted(P, lev, q.s, j)) return;
  const int64_t s = q.s;
  const double *d = dn + s;
  const double dorg = d[lamo[s + j]], tj = lamt[s + j];
  double *col = T2 + s + (s + j) * n;
  const int32_t *perm = P.w.perm + s;
  double ss = 0.0;
  for (int i = threadIdx.x; i < K; i += 256) {
    const double u = zhat[s + i] / ((d[i] - dorg) - tj);
    col[perm[i]] = u;
    ss += u * u;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  const double inv = 1.0 / sqrt((sh[0] + sh[1]) + (sh[2] + sh[3]));
  for (int i = threadIdx.x; i < K; i += 256) col[perm[i]] *= inv;
}

// Final ascending position of every eigenvalue of the merge (roots first in
// the tie order, then deflated values by index), eigenvalue output and the
// destination column of every T1 column.
__device__ void dc_final_pos(const DcProb &P, int lev, int64_t bx) {
  __shared__ double vals[256];
  const int64_t g = blockIdx.y;
  const double *dn = P.w.dn, *lamt = P.w.lamt, *ddef = P.w.ddef;
  const int32_t *cnt = P.w.cnt, *lamo = P.w.lamo;
  double *lam = P.w.lam;
  int32_t *colmap = P.w.colmap;
  const MergeGeom q = dc_geom(P.n, P.L, lev, g);
  const int64_t e = bx * blockDim.x + threadIdx.x;
  if (bx * blockDim.x >= q.m) return;
  const int64_t s = q.s;
  const int K = cnt[DC_CNT * g];
  auto val = [&](int64_t x) -> double {
    const double u = x < K ? dn[s + lamo[s + x]] + lamt[s + x] : ddef[s + (x - K)];
    if (u == u) return u;
    dc_not_a_number(P);
    return 0.0;
  };
  // ranks by counting, 256 values at a time staged in LDS (each thread looking
  // every value up for itself: 691 us a level at order 12816, this form 99)
  const double v = e < q.m ? val(e) : 0.0;
  int64_t pos = 0;
  for (int64_t x0 = 0; x0 < q.m; x0 += 256) {
    __syncthreads();
    if (x0 + threadIdx.x < q.m) vals[threadIdx.x] = val(x0 + threadIdx.x);
    __syncthreads();
    const int nx = (int)(q.m - x0 < 256 ? q.m - x0 : 256);
    const int me = (int)(e - x0 < 0 ? 0 : (e - x0 > 256 ? 256 : e - x0));   // x < e <=> x - x0 < me
    int cl = 0;
#pragma unroll 8
    for (int x = 0; x < nx; ++x) {
      const double u = vals[x];
      cl += (u < v) || (u == v && x < me);
    }
    pos += cl;
  }
  if (e >= q.m) return;
  lam[s + pos] = v;
  colmap[s + e] = (int32_t)(s + pos);
}

// nroot workgroups of weights, then the positions.
__global__ void __launch_bounds__(256) dc_lowner(const DcProb *pr, int lev, int nroot) {
  const DcProb &P = pr[blockIdx.z];
  if (lev > P.h || (int64_t)blockIdx.y >= (P.L >> lev)) return;
  const int64_t x = (int64_t)blockIdx.x - nroot;
  if (x < 0) dc_zhat(P, lev);
  else dc_final_pos(P, lev, x);
}

// Deflated columns K + 64 ch .. to their final positions, thread = row.
__device__ void dc_copy_def(const DcProb &P, int lev, int64_t rb, int64_t ch) {
  const int64_t g = blockIdx.y;
  const int64_t n = P.n, ldz = P.ldz;
  const int32_t *cnt = P.w.cnt, *colmap = P.w.colmap;
  const double *T1 = P.w.T1;
  double *Z = P.Z;
  const MergeGeom q = dc_geom(n, P.L, lev, g);
  const int64_t r = rb * blockDim.x + threadIdx.x;
  const int64_t k0 = cnt[DC_CNT * g] + ch * DC_GCOLS;
  if (r >= q.m) return;
  const int64_t k1 = k0 + DC_GCOLS < q.m ? k0 + DC_GCOLS : q.m;
#pragma unroll 8
  for (int64_t k = k0; k < k1; ++k)
    Z[(q.s + r) + (int64_t)colmap[q.s + k] * ldz] = T1[(q.s + r) + (q.s + k) * n];
}

__global__ void __launch_bounds__(GEMM_THREADS, 2) dc_gemm(const DcProb *pr, int lev, int tx, int tiles, int nrow) {
  __shared__ double lds[GEMM_LDS_DOUBLES];
  static_assert(GEMM_THREADS == 256, "shared with the row copies");
  const DcProb &P = pr[blockIdx.z];
  const int64_t g = blockIdx.y;
  if (lev > P.h || g >= (P.L >> lev)) return;
  const int64_t x = (int64_t)blockIdx.x - tiles;
  if (x >= 0) {
    dc_copy_def(P, lev, x % nrow, x / nrow);
    return;
  }
  const int64_t n = P.n, ldz = P.ldz;
  const int32_t *cnt = P.w.cnt, *colmap = P.w.colmap;
  const double *T1 = P.w.T1, *T2 = P.w.T2;
  double *Z = P.Z;
  const MergeGeom q = dc_geom(n, P.L, lev, g);
  const int K = cnt[DC_CNT * g], c1 = cnt[DC_CNT * g + 3], c12 = cnt[DC_CNT * g + 4];
  const int64_t m0 = (int64_t)(blockIdx.x % tx) * GT_M, n0 = (int64_t)(blockIdx.x / tx) * GT_N;
  if (m0 >= q.m || n0 >= K) return;
  // no column of this tile wanted (a window: the top merge is three quarters of
  // the products, 52 ms of 259 at order 12816, of which its 16 states need 16)
  {
    const int j = (int)n0 + (threadIdx.x & 63);
    if (!__any(j < K && dc_wanted(P, lev, q.s, j))) return;      // the same in every wavefront
  }
  // rows of the first child meet only kept columns [0, c12), rows of the
  // second only [c1, K); a row tile across the boundary takes all K
  int64_t k0 = 0, k1 = K;
  if (m0 + GT_M <= q.n1) k1 = c12;
  else if (m0 >= q.n1) k0 = c1;
  GemmArgs a = gemm_args(q.m, K, k1 - k0, T1 + q.s + (q.s + k0) * n, n, T2 + (q.s + k0) + q.s * n, n, Z + q.s, ldz,
                         1.0, 0.0, 0.0, 0.0);
  a.colmap = colmap + q.s;
  gemm_tile<false, A_N, B_N>(a, m0, n0, lds);
}

__global__ void dc_copy_out(const DcProb *pr) {
  const DcProb &P = pr[blockIdx.z];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P.n) P.d[i] = P.w.scl[2] == 0.0 ? P.w.lam[i] * P.w.scl[1] : NAN;
}

// ------------------------------------------------------------------ host
// Grouped divide and conquer over the table pr of `count` problems with
// orders nh[] (host copy).
int stedc_grouped(const DcProb *pr, const int64_t *nh, int64_t count, hipStream_t st) {
  if (count <= 0) return MMF_OK;
  int64_t nmax = 0;
  int hmax = 0;
  for (int64_t c = 0; c < count; ++c) {
    nmax = nh[c] > nmax ? nh[c] : nmax;
    const int h = dc_depth(nh[c]);
    hmax = h > hmax ? h : hmax;
  }
  if (nmax <= 0) return MMF_OK;
  {
    // split the batch so that merges times problems stay within 65535
    int64_t Lall = 1;
    for (int64_t c = 0; c < count; ++c) {
      const int64_t L = (int64_t)1 << dc_depth(nh[c]);
      Lall = L > Lall ? L : Lall;
    }
    const int64_t Gmax1 = Lall / 2 > 1 ? Lall / 2 : 1;
    const int64_t limit = 65535 / Gmax1;
    if (count > limit) {
      for (int64_t b = 0; b < count; b += limit) {
        const int rc = stedc_grouped(pr + b, nh + b, count - b < limit ? count - b : limit, st);
        if (rc) return rc;
      }
      return MMF_OK;
    }
  }
  const unsigned Z = (unsigned)count;
  hipLaunchKernelGGL(dc_scale, dim3(1, 1, Z), dim3(1024), 0, st, pr);
  MMF_LAUNCH_CHECK();
  hipLaunchKernelGGL(dc_tear, dim3(cdiv(nmax, 256), 1, Z), dim3(256), 0, st, pr);
  MMF_LAUNCH_CHECK();
  int64_t Lall = 0;
  for (int64_t c = 0; c < count; ++c) {
    const int64_t L = (int64_t)1 << dc_depth(nh[c]);
    Lall = L > Lall ? L : Lall;
  }
  hipLaunchKernelGGL(dc_leaf, dim3((unsigned)Lall, 1, Z), dim3(64), 0, st, pr);
  MMF_LAUNCH_CHECK();
  for (int lev = 1; lev <= hmax; ++lev) {
    int64_t Gmax = 0, maxm = 0;
    for (int64_t c = 0; c < count; ++c) {
      const int h = dc_depth(nh[c]);
      if (lev > h) continue;
      const int64_t L = (int64_t)1 << h;
      const int64_t G = L >> lev;
      const int64_t span = (int64_t)1 << lev;
      Gmax = G > Gmax ? G : Gmax;
      for (int64_t g = 0; g < G; ++g) {
        const int64_t m = dc_b((g + 1) * span, nh[c], L) - dc_b(g * span, nh[c], L);
        maxm = m > maxm ? m : maxm;
      }
    }
    if (Gmax == 0) continue;
    const unsigned nrow = cdiv(maxm, 256), nch = cdiv(maxm, DC_GCOLS), nroot = cdiv(maxm, 4);
    const unsigned tx = cdiv(maxm, GT_M), tiles = tx * cdiv(maxm, GT_N), G = (unsigned)Gmax;
    hipLaunchKernelGGL(dc_prep, dim3(nrow + nrow * cdiv(maxm, 64), G, Z), dim3(256), 0, st, pr, lev, (int)nrow);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(dc_deflate, dim3((unsigned)(Gmax * count)), dim3(64), 0, st, pr, lev, Gmax);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(dc_rotate, dim3(nrow, G, Z), dim3(256), 0, st, pr, lev);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(dc_secular, dim3(nroot + nrow * nch, G, Z), dim3(256), 0, st, pr, lev, (int)nroot, (int)nrow);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(dc_lowner, dim3(nroot + nrow, G, Z), dim3(256), 0, st, pr, lev, (int)nroot);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(dc_vectors, dim3((unsigned)maxm, G, Z), dim3(256), 0, st, pr, lev);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(dc_gemm, dim3(tiles + nrow * nch, G, Z), dim3(GEMM_THREADS), 0, st, pr, lev, (int)tx,
                       (int)tiles, (int)nrow);
    MMF_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(dc_copy_out, dim3(cdiv(nmax, 256), 1, Z), dim3(256), 0, st, pr);
  MMF_LAUNCH_CHECK();
  return MMF_OK;
}

inline DcProb dc_prob(int64_t n, double *d, const double *e, double *Z, int64_t ldz, int32_t *info,
                      const DcWs &w, const EighLimits &lim, const double *win = nullptr) {
  DcProb q;
  q.window = win != nullptr;
  q.vl = win ? win[0] : 0.0;
  q.vu = win ? win[1] : 0.0;
  q.n = n; q.ldz = ldz;
  q.sec_max = lim.secular_iters;
  q.leaf_max = lim.leaf_iters;
  q.h = dc_depth(n);
  q.L = (int64_t)1 << q.h;
  q.d = d; q.e0 = e; q.e = w.es; q.Z = Z; q.info = info;
  q.w = w;
  return q;
}

int stedc_batched(int64_t count, const int64_t *n, double *const *d, double *const *e, double *const *Z,
                  const int64_t *ldz, void *const *stage, int32_t *const *info, void *table, hipStream_t st,
                  const EighLimits &lim) {
  static_assert(sizeof(DcProb) <= STAGE_TABLE_BYTES, "table entry");
  std::vector<DcProb> h((size_t)count);
  for (int64_t c = 0; c < count; ++c)
    h[c] = dc_prob(n[c], d[c], e[c], Z[c], ldz[c], info[c], stedc_ws(n[c], (char *)stage[c] + 512), lim);
  DcProb *pr = reinterpret_cast<DcProb *>(table);
  const int rc = table_write(pr, h.data(), count, st);
  if (rc) return rc;
  return stedc_grouped(pr, n, count, st);
}

int stedc_run(int64_t n, double *d, const double *e, double *Z, int64_t ldz, void *work, size_t bytes,
              int32_t *info, hipStream_t st, const EighLimits &lim, const double *win) {
  if (n <= 0) return MMF_OK;
  static_assert(sizeof(DcProb) <= 512, "table entry");
  DcWs w = stedc_ws(n, (char *)work + 512);
  if (bytes < w.bytes + 512) return MMF_ERR_WORKSPACE;
  DcProb *pr = reinterpret_cast<DcProb *>(work);
  const DcProb q = dc_prob(n, d, e, Z, ldz, info, w, lim, win);
  const int rc = table_write(pr, &q, 1, st);
  if (rc) return rc;
  return stedc_grouped(pr, &n, 1, st);
}

}  // namespace mmf

using namespace mmf;

extern "C" int mmf_stedc(int64_t n, double *d, const double *e, double *Z, int64_t ldz, void *work,
                         size_t work_bytes, int32_t *dev_info, void *stream) {
  if (n < 0) return -1;
  if (!d) return -2;
  if (n > 1 && !e) return -3;
  if (!Z) return -4;
  if (ldz < n || ldz < 1) return -5;
  if (!work) return -6;
  if (work_bytes < stedc_ws_bytes(n)) return -7;
  if (!dev_info) return -8;
  return stedc_run(n, d, e, Z, ldz, work, work_bytes, dev_info, (hipStream_t)stream);
}
