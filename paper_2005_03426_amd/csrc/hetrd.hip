// Blocked Householder reduction of a complex Hermitian matrix to a real
// symmetric tridiagonal matrix (stage 1 of the dense eigensolve that the
// paper delegates to LAPACK, Sec. 3.2).
//
// Q^H A Q = T,  Q = H_0 H_1 ... H_{n-2},  H_i = I - tau_i v_i v_i^H,
// v_i = (0,..,0, 1, x/(alpha - beta)) with beta = -sign(Re alpha) ||(alpha, x)||
// real, so T is real: d_i = Re a_ii, e_i = beta_i.
//
// Panels of HT_NB columns.  Inside a panel, column i = p + k is reduced
// against the *unupdated* trailing matrix: with V, W the panel's previous
// reflectors and their companions, the current trailing matrix is
// A - V W^H - W V^H, so
//   u = A v - V (W^H v) - W (V^H v),   w0 = tau u,   w = w0 - (tau/2)(w0^H v) v.
// After the panel the trailing matrix takes one rank-2k update
// A -= [V W] [W V]^H on the matrix cores (lower triangle only).
//
// Per column two launches (the order of the reduction is a chain of n - 1
// columns, so below a few thousand rows its time is launches and dependent
// memory round trips, not bytes):
//   ht_column: every workgroup derives (beta, tau, scale) from the raw column
//     x and its norm partials, forms the entries of v it needs from x, and
//     does its share of A v over the lower trailing triangle, of v^H A v, of
//     the panel products W^H v / V^H v, or stores v;
//   ht_finish: u from the partials.  With x1 = W^H v, x2 = V^H v,
//     v^H u = v^H A v - 2 Re(x2^H x1) =: g is real, so w = tau u - (|tau|^2 g
//     / 2) v needs no further pass over the rows; the same launch updates
//     column i+1 by the k+1 reflectors so far (w[i+1] formed in every
//     workgroup) and leaves its norm partials.
// Four launches per column (reflector, product, u, w with the next column)
// took 18.5 us per column at order 82, 23 at 450 and 31.5 at 1715
// (profiled); the two take 2.1 (all in the tail), 10.0 and 11.5.  (The figures
// beside the single choices below are those of the change that made them; whole
// solves take 4.9 ms at order 450 in the dressed basis, 21.2 at 1715 and 138 at
// 5000 with all of them.)
// The last HT_TAIL rows of every matrix (all of a smaller one) are reduced by
// one workgroup in registers (ht_tail).
// All sums are over fixed partitions in fixed order (deterministic).
//
// Every kernel is a template over the scalar type R: R = double is the
// complex128 path; R = float is the complex64 reduction of the precision
// layer (FP32 storage, FP32 accumulation, FP32 matrix cores), whose d and e
// are still returned in FP64.
//
// Grouped execution: every kernel takes a device table of problems (HtProb)
// and works on problem blockIdx.z, so one launch advances column i of every
// matrix of a batch; a matrix that has reached its tail simply exits.  Grids are sized for the largest matrix.  A single reduction is the
// one-entry case.
#include <vector>
#include "common.h"
#include "stages.h"
#include "gemm_core.h"
#include "ktimer.h"
#include "table.h"

namespace mmf {

constexpr int HV_T = 64;        // HEMV tile
constexpr int HV_CH = 8;        // most interior tiles per HEMV workgroup (one block column strip)
constexpr int64_t HV_NT_BYTES = (int64_t)512 << 20;   // lower trailing triangle from which its tiles are read non-temporally
constexpr int DOT_MIN = 256;    // fewest rows per wavefront of the panel dot products
constexpr int HT_TAIL = 128;    // largest order of the register tail: 32 entries a lane
constexpr int TAIL_THREADS = 512;

// First column of the tail: the panels before it are all full.
__host__ __device__ inline int64_t ht_tail_start(int64_t n) {
  return n <= HT_TAIL ? 0 : (n - HT_TAIL + HT_NB - 1) / HT_NB * HT_NB;
}

template <typename R>
struct HtWs {
  cx<R> *P3;       // n x 3NB (ld n): [V | W | V]
  cx<R> *x;        // mpad: the current column before it is scaled into v
  cx<R> *pdir;     // nbt x mpad: direct partial of block column lb for local row
  cx<R> *ptrn;     // nbt x nchmax x 64: transposed partials (slots 0, 1: diagonal, edge tile)
  cx<R> *dots;     // gdot x 2NB
  R *norms;        // nbt partials
  R *sparts;       // nbt x nchmax partials of v^H A v
  int64_t nbt, mpad, nchmax;
  size_t bytes;
};

template <typename R>
inline HtWs<R> hetrd_ws(int64_t n, void *base) {
  Carver cv(base);
  HtWs<R> w;
  // HEMV tiles sit on the absolute 64-row grid of A: block columns of the
  // trailing matrix number at most ceil(n / 64)
  w.nbt = (n + HV_T - 1) / HV_T;
  if (w.nbt < 1) w.nbt = 1;
  w.mpad = w.nbt * HV_T;
  w.nchmax = w.nbt + 2;                          // one interior tile per workgroup at least
  w.P3 = cv.take<cx<R>>((size_t)n * 3 * HT_NB);
  w.x = cv.take<cx<R>>((size_t)w.mpad);
  w.pdir = cv.take<cx<R>>((size_t)w.nbt * w.mpad);
  w.ptrn = cv.take<cx<R>>((size_t)w.nbt * w.nchmax * HV_T);
  const int64_t gdot = (n + DOT_MIN - 1) / DOT_MIN + 1;
  w.dots = cv.take<cx<R>>((size_t)gdot * 2 * HT_NB);
  w.norms = cv.take<R>((size_t)w.nbt + 1);
  w.sparts = cv.take<R>((size_t)w.nbt * w.nchmax);
  w.bytes = cv.used();
  return w;
}

template <typename R>
size_t hetrd_ws_bytes_t(int64_t n) { return hetrd_ws<R>(n, nullptr).bytes; }
size_t hetrd_ws_bytes(int64_t n) { return hetrd_ws_bytes_t<double>(n) + 256; }

// Split of one matrix's sums, from its own order and the panel alone (a
// matrix gives the same bits alone and in any batch).
// Interior tiles per workgroup of the panel at column p: at most 128
// workgroups of single tiles, then strips of up to HV_CH (the next tile is
// loaded during the current one).  Strips of eight at every order left 200 of
// the 256 CUs idle at order 1715 (17.7 us per product against 6.9 for single
// tiles).  Targets of 512 / 256 / 128 / 64 workgroups: order 1715 alone 31.0 /
// 31.2 / 31.2 / 33.1 ms, 48 uneven matrices together, which fill the chip
// anyway, 151 / 147 / 140 / 135 ms, order 5000 180 / 177 / 181 / 184 ms.
__host__ __device__ inline int ht_strip(int64_t n, int64_t p) {
  const int64_t nb = n / HV_T - (p + 1) / HV_T;
  const int64_t want = (nb * (nb - 1) / 2 + 127) / 128;
  return (int)(want < 1 ? 1 : (want > HV_CH ? HV_CH : want));
}
// Strips of local block column lb of column i's trailing matrix.
__host__ __device__ inline int ht_strips(int64_t n, int64_t i, int ch, int64_t lb) {
  const int64_t inner = n / HV_T - (i + 1) / HV_T - lb - 1;
  return inner > 0 ? (int)((inner + ch - 1) / ch) : 0;
}
// Rows per wavefront of the panel products: one round of four loads per lane
// while the partials stay few, longer chunks for long columns.
__host__ __device__ inline int ht_dot_rows(int64_t n) { return n <= 8 * DOT_MIN ? DOT_MIN : 4 * DOT_MIN; }

// one row of the problem table
template <typename R>
struct HtProb {
  int64_t n, lda, mpad, nchmax;
  cx<R> *A;
  double *d, *e;
  cx<R> *tau;
  cx<R> *P3, *x, *pdir, *ptrn, *dots;
  R *norms, *sparts;
};

template <typename R>
inline HtProb<R> ht_prob(int64_t n, cx<R> *A, int64_t lda, double *d, double *e, cx<R> *tau,
                         const HtWs<R> &w) {
  HtProb<R> q;
  q.n = n; q.lda = lda; q.mpad = w.mpad; q.nchmax = w.nchmax;
  q.A = A; q.d = d; q.e = e; q.tau = tau;
  q.P3 = w.P3; q.x = w.x; q.pdir = w.pdir; q.ptrn = w.ptrn; q.dots = w.dots;
  q.norms = w.norms; q.sparts = w.sparts;
  return q;
}

// ---------------------------------------------------------------- kernels
// First column of a panel: x <- A[p:, p], d[p], and the partial norms of
// x[p+2:] per 64-row block of the absolute grid (one wavefront each).
template <typename R>
__global__ void __launch_bounds__(256) ht_colnorm(const HtProb<R> *pr, int64_t p) {
  const HtProb<R> &q = pr[blockIdx.z];
  const int64_t n = q.n;
  if (p >= ht_tail_start(n)) return;
  const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);     // local block
  const int64_t r = (p / HV_T + blk) * HV_T + (threadIdx.x & 63);
  if ((p / HV_T + blk) * HV_T >= n) return;                             // wavefront-uniform
  cx<R> a = cmk<R>(0, 0);
  if (r >= p && r < n) {
    a = gload((const MMF_GLOBAL cx<R> *)q.A + r + p * q.lda);
    ((MMF_GLOBAL cx<R> *)q.x)[r] = a;
    if (r == p) q.d[p] = (double)a.re;
  }
  const R s = wave_sum(r >= p + 2 ? cabs2(a) : R(0));
  if ((threadIdx.x & 63) == 0) q.norms[blk] = s;
}

// Householder scalars of a column (alpha, x) with |x|^2 = xn2: the real beta,
// tau and scale = 1 / (alpha - beta) with v = (1, scale x).
template <typename R>
__device__ __forceinline__ void ht_scalars(cx<R> alpha, R xn2, R &beta, cx<R> &tau, cx<R> &scale) {
  if (xn2 == R(0) && alpha.im == R(0)) {
    beta = alpha.re;
    tau = cmk<R>(0, 0);
    scale = cmk<R>(0, 0);
  } else {
    const R nrm = sqrt(alpha.re * alpha.re + alpha.im * alpha.im + xn2);
    beta = alpha.re >= R(0) ? -nrm : nrm;
    tau = cmk<R>((beta - alpha.re) / beta, -alpha.im / beta);
    const cx<R> den = cmk<R>(alpha.re - beta, alpha.im);
    const R q = den.re * den.re + den.im * den.im;
    scale = cmk<R>(den.re / q, -den.im / q);
  }
}

// The same of column i from its norm partials (one per 64-row block from row i on), in every lane.
template <typename R>
__device__ __forceinline__ void ht_column_scalars(const HtProb<R> &q, int64_t i, R &beta, cx<R> &tau, cx<R> &scale) {
  const MMF_GLOBAL R *norms = (const MMF_GLOBAL R *)q.norms;
  const int cnt = (int)((q.n + HV_T - 1) / HV_T - i / HV_T);
  const cx<R> alpha = gload((const MMF_GLOBAL cx<R> *)q.x + i + 1);
  R s = 0;
  for (int g = threadIdx.x & 63; g < cnt; g += 64) s += norms[g];
  ht_scalars<R>(alpha, wave_sum(s), beta, tau, scale);
}

// v[r] of column i from the raw column's entry xr
template <typename R>
__device__ __forceinline__ cx<R> ht_v(cx<R> xr, int64_t r, int64_t i, int64_t n, cx<R> scale) {
  const cx<R> v = cmul(xr, scale);
  return (r <= i || r >= n) ? cmk<R>(0, 0) : (r == i + 1 ? cmk<R>(1, 0) : v);
}

// d += a vc and t += conj(at) vr (at = a, or zero on the diagonal) in fused
// operations: the same bits in every form of the product
template <typename R>
__device__ __forceinline__ void ht_tile_fma(cx<R> a, cx<R> at, cx<R> vc, cx<R> vr, cx<R> &d, cx<R> &t) {
  d.re = fma(a.re, vc.re, d.re);
  d.re = fma(-a.im, vc.im, d.re);
  d.im = fma(a.re, vc.im, d.im);
  d.im = fma(a.im, vc.re, d.im);
  t.re = fma(at.re, vr.re, t.re);
  t.re = fma(at.im, vr.im, t.re);
  t.im = fma(at.re, vr.im, t.im);
  t.im = fma(-at.im, vr.re, t.im);
}

template <typename R> struct NtVec;
template <> struct NtVec<double> { typedef double v __attribute__((ext_vector_type(2))); };
template <> struct NtVec<float> { typedef float v __attribute__((ext_vector_type(2))); };

// Panel products of column i for row chunk g (dr rows):
// dots[g*2NB + q] = sum conj(W[:,q]) v and dots[g*2NB + NB + q] =
// sum conj(V[:,q]) v (q < k) over its rows of [i+1, n).  One wavefront per
// product qq (lane l sums rows l, l + 64, ...), from x: v = scale x below row
// i + 1, so that the reads need not wait for the column's scalars (order 450 4.90
// -> 4.83 ms, 5000 140.9 -> 137.2, 48 uneven ones 110.1 -> 108.9).
template <typename R>
__device__ void ht_dots_wave(const HtProb<R> &pq, int64_t i, int k, int g, int qq, int dr) {
  const int64_t n = pq.n;
  const int q = qq % k, which = qq / k;
  const MMF_GLOBAL cx<R> *X = (const MMF_GLOBAL cx<R> *)pq.P3 + (int64_t)(which == 0 ? HT_NB + q : q) * n;
  const MMF_GLOBAL cx<R> *x = (const MMF_GLOBAL cx<R> *)pq.x;
  const int lane = threadIdx.x & 63;
  const int64_t r0 = i + 1 + (int64_t)g * dr;
  cx<R> s = cmk<R>(0, 0), first = s;
  for (int j0 = 0; j0 < dr && r0 + j0 < n; j0 += 256) {
    cx<R> a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t r = r0 + j0 + 64 * u + lane, rc = r < n ? r : n - 1;
      a[u] = gload(X + rc);
      b[u] = gload(x + rc);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t r = r0 + j0 + 64 * u + lane;
      const bool on = r < n && r > i + 1;
      s = cadd(s, cmulc(a[u], cmk<R>(on ? b[u].re : R(0), on ? b[u].im : R(0))));
      if (r == i + 1) first = cconj(a[u]);          // v is one there
    }
  }
  R beta;
  cx<R> tau, scale;
  ht_column_scalars<R>(pq, i, beta, tau, scale);
  s = cadd(cmul(scale, s), first);
  const R re = wave_sum(s.re), im = wave_sum(s.im);
  if (lane == 0) ((MMF_GLOBAL cx<R> *)pq.dots)[(int64_t)g * 2 * HT_NB + which * HT_NB + q] = cmk<R>(re, im);
}

// u = A_trail v over the lower triangle of the trailing matrix
// A_trail = A[i+1:, i+1:].  Tiles lie on the absolute 64 x 64 grid of A
// (block b covers rows 64b .. 64b+63), so on a leading dimension divisible by
// 8 every column segment a load touches starts on a 128-byte line; b0 is the
// block holding row i+1 and local block lb = b - b0.  Work items:
//   blockIdx.y < strip_rows: the strips of `ch` interior tiles, block columns
//     x and nbl - 1 - x one after the other (the triangle folded, so that few
//     workgroups are empty);
//   the others, in a row: the diagonal tiles (slot 0; masked: lower triangle,
//     real diagonal; they also store v of their rows), the tiles in the last
//     block row when that is partial (slot 1), the panel products.
// (One workgroup per block column and slot of the widest one, and per block
// column and product, left three of four empty: 20 matrices of order 1900
// took 127 ms against 120 now, 48 of order 900 48 against 43.)
// The four wavefronts share every tile, wave w taking its columns
// 16w .. 16w+15 (lane: rows rg + 16q, columns 16w + 4cg + j), so a lane holds
// 16 elements per tile; the next tile is loaded while the current one is
// multiplied, and the first one before the column's scalars are known.  The
// direct product is summed over the waves through LDS once per tile and
// written as the partial of (block column, row); the conjugate-transposed
// product stays in registers over the strip.  Columns left of i+1 carry v = 0.
// Bound: HBM at large orders; below about 3000 rows, where the strips of one
// tile leave no second tile to overlap with, one launch's dependent loads.
// Without STRIP (every matrix of the launch has single-tile strips) all tiles
// take the masked form, which needs no second tile's registers (145 against
// 240) and loads x ahead too.  With the wide ht_finish: order 450 6.07 -> 5.55
// ms, 1715 24.8 -> 22.5 ms, 5000 155.4 -> 149.8 ms, 48 matrices 128.2 -> 125.1
// ms (whole calls).
// NT: the tiles are read non-temporally, so that a triangle far larger than
// the 256 MB last-level cache does not sweep everything else out of it.  With
// ordinary reads the reduction takes 26.7 ms against 28.5 at order 2048, 84.0
// against 93.3 at 4000, 184.5 against 203.4 at 6000, 389.8 against 396.2 at
// 8000, but 947.6 against 897.3 at 11000: NT above HV_NT_BYTES.
template <typename R, bool NT, bool STRIP>
__global__ void __launch_bounds__(256, 2) ht_column(const HtProb<R> *pr, int64_t p, int k, int strip_rows) {
  typedef cx<R> C;
  typedef typename NtVec<R>::v nv;
  __shared__ C red[2][4][HV_T];
  __shared__ R shs[4];
  const HtProb<R> &q = pr[blockIdx.z];
  const int64_t n = q.n, lda = q.lda, mpad = q.mpad, nchmax = q.nchmax, i = p + k;
  if (p >= ht_tail_start(n)) return;
  const int ch = ht_strip(n, p), dr = ht_dot_rows(n);
  const int64_t b0 = (i + 1) / HV_T;
  const int64_t nb = (n + HV_T - 1) / HV_T;        // absolute blocks
  const int64_t nfull = n / HV_T;                   // blocks entirely inside the matrix
  const int nbl = (int)(nb - b0);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  int lb, slot;
  int64_t first;                                    // first tile's block row
  if ((int)blockIdx.y < strip_rows) {
    lb = blockIdx.x;
    if (2 * lb > nbl - 1) return;
    int c = blockIdx.y;
    const int c0 = ht_strips(n, i, ch, lb);
    if (c >= c0) {
      c -= c0;
      const int other = nbl - 1 - lb;
      if (other == lb || c >= ht_strips(n, i, ch, other)) return;
      lb = other;
    }
    slot = 2 + c;
    first = b0 + lb + 1 + (int64_t)c * ch;
  } else {
    int item = ((int)blockIdx.y - strip_rows) * (int)gridDim.x + (int)blockIdx.x;
    const bool edge = nb != nfull;
    if (item >= 2 * nbl) {                          // panel products of this column
      item -= 2 * nbl;
      const int chunks = (int)((n - i - 1 + dr - 1) / dr);
      const int qq = item / chunks * 4 + wave;
      if (qq < 2 * k) ht_dots_wave(q, i, k, item % chunks, qq, dr);
      return;
    }
    slot = item >= nbl;
    lb = slot ? item - nbl : item;
    first = slot ? nb - 1 : b0 + lb;
    if (slot && (!edge || lb == nbl - 1)) {         // its partial of v^H A v is summed all the same
      if (tid == 0) q.sparts[lb * nchmax + 1] = R(0);
      return;
    }
  }
  const int64_t bj = b0 + lb;
  const MMF_GLOBAL C *A = (const MMF_GLOBAL C *)q.A;
  const MMF_GLOBAL C *x = (const MMF_GLOBAL C *)q.x;
  MMF_GLOBAL C *pdir = (MMF_GLOBAL C *)q.pdir, *ptrn = (MMF_GLOBAL C *)q.ptrn;
  const int rg = lane & 15, cg = lane >> 4;
  const int cb = 16 * wave + 4 * cg;
  const int64_t col0 = bj * HV_T + cb;
  C vc[4], tacc[4];
  R beta, gpart = 0;
  C tau, scale;
  if (!STRIP || slot < 2) {
    // ------------------------------------------------ one tile, masked; its
    // entries and the raw x of its rows and columns before the scalars
    const int64_t row0 = first * HV_T + rg;
    C a[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const int64_t row = row0 + 16 * qq, col = col0 + j;
        const bool ok = row < n && row >= col;
        const C t = gload(A + (ok ? row + col * lda : 0));
        a[j][qq] = cmk<R>(ok ? t.re : R(0), ok && row != col ? t.im : R(0));
      }
    C vr[4], dacc[4];
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
      vr[qq] = gload(x + row0 + 16 * qq);
      vc[qq] = gload(x + col0 + qq);
    }
    ht_column_scalars<R>(q, i, beta, tau, scale);
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
      vr[qq] = ht_v<R>(vr[qq], row0 + 16 * qq, i, n, scale);
      dacc[qq] = cmk<R>(0, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      vc[j] = ht_v<R>(vc[j], col0 + j, i, n, scale);
      tacc[j] = cmk<R>(0, 0);
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const bool dg = row0 + 16 * qq == col0 + j;
        ht_tile_fma<R>(a[j][qq], dg ? cmk<R>(0, 0) : a[j][qq], vc[j], vr[qq], dacc[qq], tacc[j]);
        gpart += dg ? a[j][qq].re * cabs2(vr[qq]) : R(0);
      }
    }
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
      const R re = rows_sum(dacc[qq].re), im = rows_sum(dacc[qq].im);
      if (cg == 0) red[0][wave][rg + 16 * qq] = cmk<R>(re, im);
    }
    __syncthreads();
    if (tid < HV_T) {
      pdir[lb * mpad + (first - b0) * HV_T + tid] =
          cadd(cadd(red[0][0][tid], red[0][1][tid]), cadd(red[0][2][tid], red[0][3][tid]));
      const int64_t r = bj * HV_T + tid;
      if (slot == 0 && r > i && r < n) {            // this block's rows of v
        const C v = ht_v<R>(gload(x + r), r, i, n, scale);
        MMF_GLOBAL C *P3 = (MMF_GLOBAL C *)q.P3;
        ((MMF_GLOBAL C *)q.A)[r + i * lda] = v;
        P3[r + (int64_t)k * n] = v;
        P3[r + (int64_t)(2 * HT_NB + k) * n] = v;
        if (r == i + 1) {
          q.e[i] = (double)beta;
          q.tau[i] = tau;
        }
      }
    }
  } else {
    // -------------------------------------------------- interior strip
    const int64_t bi1 = (first + ch < nfull) ? first + ch : nfull;
    const MMF_GLOBAL C *colp = A + col0 * lda + rg;
    C b0t[4][4], b1t[4][4];
    auto load = [&](C (&b)[4][4], int64_t bi) {
      const MMF_GLOBAL C *p = colp + bi * HV_T;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          const MMF_GLOBAL nv *at = reinterpret_cast<const MMF_GLOBAL nv *>(p + 16 * qq + (int64_t)j * lda);
          const nv y = NT ? __builtin_nontemporal_load(at) : *at;
          b[j][qq] = cmk<R>(y[0], y[1]);
        }
    };
    auto step = [&](C (&b)[4][4], C (&nxt)[4][4], int64_t bi, int t) {
      if (bi + 1 < bi1) load(nxt, bi + 1);
      __builtin_amdgcn_sched_barrier(0);
      C vr[4], dacc[4];
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        vr[qq] = cmul(gload(x + bi * HV_T + rg + 16 * qq), scale);   // rows of an interior tile are below i + 1
        dacc[qq] = cmk<R>(0, 0);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          ht_tile_fma<R>(b[j][qq], b[j][qq], vc[j], vr[qq], dacc[qq], tacc[j]);
        }
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const R re = rows_sum(dacc[qq].re), im = rows_sum(dacc[qq].im);
        if (cg == 0) red[t & 1][wave][rg + 16 * qq] = cmk<R>(re, im);
      }
      __syncthreads();
      if (tid < HV_T) {
        const C s = cadd(cadd(red[t & 1][0][tid], red[t & 1][1][tid]), cadd(red[t & 1][2][tid], red[t & 1][3][tid]));
        pdir[lb * mpad + (bi - b0) * HV_T + tid] = s;
      }
    };
    load(b0t, first);
    __builtin_amdgcn_sched_barrier(0);
    ht_column_scalars<R>(q, i, beta, tau, scale);
#pragma unroll
    for (int j = 0; j < 4; ++j) { vc[j] = ht_v<R>(gload(x + col0 + j), col0 + j, i, n, scale); tacc[j] = cmk<R>(0, 0); }
    int t = 0;
    for (int64_t bi = first; bi < bi1; bi += 2, t += 2) {
      step(b0t, b1t, bi, t);
      if (bi + 1 < bi1) step(b1t, b0t, bi + 1, t + 1);
    }
  }
  // transposed partial (the same in the 16 lanes of a column group) and this
  // strip's part of v^H A v: 2 Re(v_J^H tacc), plus the real diagonal
  R gt = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const R re = row16_sum(tacc[j].re), im = row16_sum(tacc[j].im);
    if (rg == j) ptrn[(lb * nchmax + slot) * HV_T + cb + j] = cmk<R>(re, im);
    gt += vc[j].re * re + vc[j].im * im;
  }
  const R gw = 2 * rows_sum(gt) + wave_sum(gpart);
  if (lane == 0) shs[wave] = gw;
  __syncthreads();
  if (tid == 0) q.sparts[lb * nchmax + slot] = (shs[0] + shs[1]) + (shs[2] + shs[3]);
}

// get(0) + ... + get(min(last, N - 1)), all N entries read before the first is
// added: a loop's remainder waits for memory once per entry (order 1715 21.56
// -> 21.21 ms, refined 1352 18.46 -> 18.15; eight at once: 450 1 % slower).
constexpr int HF_LOADS = 4;
template <int N, typename Get>
__device__ __forceinline__ auto ht_sum_ahead(Get get, int last) {
  if (last <= 0) return get(0);
  decltype(get(0)) t[N];
#pragma unroll
  for (int j = 0; j < N; ++j) t[j] = get(j);
#pragma unroll
  for (int j = 1; j < N; ++j) {
    t[j].re = j <= last ? t[j].re : 0;
    t[j].im = j <= last ? t[j].im : 0;
  }
#pragma unroll
  for (int w = N / 2; w > 0; w /= 2)
#pragma unroll
    for (int j = 0; j < w; ++j) t[j] = cadd(t[j], t[j + w]);
  return t[0];
}

// Column i = p + k after ht_column: w = tau u - (|tau|^2 g / 2) v, and inside
// the panel column i+1 updated by the k+1 reflectors so far.  One workgroup
// per 64-row block.  Parts 0 .. 3 (a wavefront each) split the partial sums
// and the panel columns (each V, W entry is read once for both corrections),
// combined in LDS in fixed order; 4 sums the panel products, 5 and 6 the
// partials of v^H A v, 7 forms w[i+1].
// Latency bound (table, partials, stores, two barriers), so with WIDE the sums
// that feed the scalars run beside the row sums, in eight wavefronts: 4.9 us
// at order 1715 against 6.3 in four wavefronts that each take two parts.  Above
// two workgroups per CU the narrow form is the faster one; both give the same
// bits.  Eigenvalues with the line at 256, 512, 1024 workgroups: 20 x 1900 117.6,
// 116.9, 117.1 ms; 48 x 900 41.8, 41.3, 41.7; 48 x 450 12.2, 11.9, 12.0; 200 x 300
// 11.8, 11.6, 11.9.
constexpr int64_t HF_WIDE_MAX = 512;              // most workgroups of a launch in the wide form
template <typename R, bool WIDE>
__global__ void __launch_bounds__(WIDE ? 512 : 256) ht_finish(const HtProb<R> *pr, int64_t p, int k) {
  typedef cx<R> C;
  constexpr int QW = HT_NB / 4;
  __shared__ C x1[HT_NB], x2[HT_NB], cw[HT_NB], cv[HT_NB];
  __shared__ C part[4][HV_T], apart[4][HV_T];
  __shared__ R sh[2], xxs;
  __shared__ C w1s;
  const HtProb<R> &pq = pr[blockIdx.z];
  const int64_t n = pq.n, lda = pq.lda, mpad = pq.mpad, nchmax = pq.nchmax, i = p + k;
  if (p >= ht_tail_start(n)) return;
  const int ch = ht_strip(n, p), dr = ht_dot_rows(n);
  const int64_t b0 = (i + 1) / HV_T;
  const int64_t nb = (n + HV_T - 1) / HV_T, nfull = n / HV_T;
  const int64_t lbi = blockIdx.x;                   // local block of these rows
  if (b0 + lbi >= nb) return;                       // beyond this matrix's blocks
  MMF_GLOBAL C *P3 = (MMF_GLOBAL C *)pq.P3;
  const MMF_GLOBAL C *pdir = (const MMF_GLOBAL C *)pq.pdir, *ptrn = (const MMF_GLOBAL C *)pq.ptrn;
  const MMF_GLOBAL C *dots = (const MMF_GLOBAL C *)pq.dots;
  const MMF_GLOBAL R *sparts = (const MMF_GLOBAL R *)pq.sparts;
  const bool next = k + 1 < HT_NB;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int64_t rho = (b0 + lbi) * HV_T + lane;     // absolute row
  const bool live = rho > i && rho < n;
  const C tau = gload((const MMF_GLOBAL C *)pq.tau + i);
  C vq[QW], wq[QW], u = cmk<R>(0, 0), v = cmk<R>(0, 0), a = cmk<R>(0, 0), r1 = cmk<R>(0, 0);
  const int part2 = WIDE ? wave : wave + 4;         // 4 .. 7: the second part of this wavefront
  if (wave < 4) {
    // ---- V, W of this row, the partials of u
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      const int qc = wave + 4 * j;
      vq[j] = wq[j] = cmk<R>(0, 0);
      if (qc < k && live) {
        vq[j] = gload(P3 + rho + (int64_t)qc * n);
        wq[j] = gload(P3 + rho + (int64_t)(HT_NB + qc) * n);
      }
    }
    if (wave == 0 && live) {
      v = gload(P3 + rho + (int64_t)k * n);
      if (next) a = gload((const MMF_GLOBAL C *)pq.A + rho + (i + 1) * lda);
    }
    // direct partials of block columns wave, wave + 4, ..., transposed partials
    // of this block column's slots (beyond the last one it is read again for nothing)
    const MMF_GLOBAL C *pc = pdir + lbi * HV_T + lane;
    for (int64_t l0 = wave; l0 <= lbi; l0 += 4 * HF_LOADS)
      u = cadd(u, ht_sum_ahead<HF_LOADS>([&](int j) {
        const int64_t lb = l0 + 4 * j;
        return gload(pc + (lb < lbi ? lb : lbi) * mpad);
      }, (int)((lbi - l0) >> 2)));
    const int nin = ht_strips(n, i, ch, lbi);
    const bool edge = nb != nfull && b0 + lbi < nb - 1;
    const MMF_GLOBAL C *pt = ptrn + lbi * nchmax * HV_T + lane;
    for (int c0 = wave; c0 < nin; c0 += 4 * HF_LOADS)
      u = cadd(u, ht_sum_ahead<HF_LOADS>([&](int j) {
        const int c = c0 + 4 * j;
        return gload(pt + (int64_t)((c < nin ? c : nin - 1) + 2) * HV_T);
      }, (nin - 1 - c0) >> 2));
    if (wave == 1) u = cadd(u, gload(pt));
    if (wave == 2 && edge) u = cadd(u, gload(pt + HV_T));
  }
  if (part2 == 4) {
    // ---- panel products x1 (lanes < k), x2 (the next k) and 2 Re(x2^H x1)
    const int gdot = (int)((n - i - 1 + dr - 1) / dr);
    C s = cmk<R>(0, 0);
    const bool on = lane < 2 * k;
    const int qc = lane < k ? lane : lane - k;
    if (on) {
      const MMF_GLOBAL C *dp = dots + (lane < k ? 0 : HT_NB) + qc;
      for (int g0 = 0; g0 < gdot; g0 += HF_LOADS)
        s = cadd(s, ht_sum_ahead<HF_LOADS>([&](int j) {
          return gload(dp + (int64_t)(g0 + j < gdot ? g0 + j : gdot - 1) * 2 * HT_NB);
        }, gdot - 1 - g0));
      if (lane < k) x1[qc] = s; else x2[qc] = s;
    }
    const R ore = __shfl(s.re, (lane + k) & 63, 64), oim = __shfl(s.im, (lane + k) & 63, 64);
    const R xx = wave_sum(lane < k ? s.re * ore + s.im * oim : R(0));
    if (lane == 0) xxs = xx;
  } else if (part2 == 5 || part2 == 6) {
    // ---- v^H A v
    const int nbl = (int)(nb - b0), t = (part2 - 5) * 64 + lane;
    R s = 0;
    for (int lb = t >> 3; lb < nbl; lb += 16) {
      const int nsl = 2 + ht_strips(n, i, ch, lb);
#pragma unroll 4
      for (int c = t & 7; c < nsl; c += 8) s += gload(sparts + lb * nchmax + c);
    }
    s = wave_sum(s);
    if (lane == 0) sh[part2 - 5] = s;
  } else if (part2 == 7) {
    // ---- row i+1 of the partials and of V, W
    const int row = (int)(i + 1 - b0 * HV_T);
    const int nin = ht_strips(n, i, ch, 0);
    const bool edge = nb != nfull && b0 < nb - 1;
    if (lane < k) {
      cv[lane] = cconj(gload(P3 + (i + 1) + (int64_t)lane * n));
      cw[lane] = cconj(gload(P3 + (i + 1) + (int64_t)(HT_NB + lane) * n));
    }
    for (int c = lane; c < nin; c += 64) r1 = cadd(r1, gload(ptrn + (int64_t)(c + 2) * HV_T + row));
    if (lane == 0) r1 = cadd(r1, cadd(gload(pdir + row), gload(ptrn + row)));
    if (lane == 1 && edge) r1 = cadd(r1, gload(ptrn + HV_T + row));
  }
  __syncthreads();
  // ---- alpha = -|tau|^2 g / 2 with g = v^H A v - 2 Re(x2^H x1)
  const R alpha = R(-0.5) * cabs2(tau) * ((sh[0] + sh[1]) - 2 * xxs);
  if (wave < 4) {
    C as = cmk<R>(0, 0);
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      const int qc = wave + 4 * j;
      if (qc < k) {
        u = csub(u, cmul(vq[j], x1[qc]));
        u = csub(u, cmul(wq[j], x2[qc]));
        as = cadd(as, cmul(vq[j], cw[qc]));
        as = cadd(as, cmul(wq[j], cv[qc]));
      }
    }
    part[wave][lane] = u;
    apart[wave][lane] = as;
  }
  if (part2 == 7) {                                 // w[i+1] = tau u[i+1] + alpha (v[i+1] = 1)
    if (lane < k) {
      r1 = csub(r1, cmul(cconj(cv[lane]), x1[lane]));
      r1 = csub(r1, cmul(cconj(cw[lane]), x2[lane]));
    }
    const C us = cmk<R>(wave_sum(r1.re), wave_sum(r1.im));
    const C w0 = cmul(tau, us);
    if (lane == 0) w1s = cmk<R>(w0.re + alpha, w0.im);
  }
  __syncthreads();
  if (wave != 0) return;
  R nrm = 0;
  if (live) {
    const C us = cadd(cadd(part[0][lane], part[1][lane]), cadd(part[2][lane], part[3][lane]));
    const C w1 = w1s;
    C w = cadd(cmul(tau, us), cscale(v, alpha));
    if (rho == i + 1) w = w1;
    P3[rho + (int64_t)(HT_NB + k) * n] = w;
    if (next) {
      a = csub(a, cadd(cadd(apart[0][lane], apart[1][lane]), cadd(apart[2][lane], apart[3][lane])));
      a = csub(a, cadd(cmul(v, cconj(w1)), w));     // conj(v[i+1]) = 1
      ((MMF_GLOBAL C *)pq.x)[rho] = a;
      if (rho == i + 1) pq.d[i + 1] = (double)a.re;
      if (rho >= i + 3) nrm = cabs2(a);
    }
  }
  if (next) {
    nrm = wave_sum(nrm);
    // ht_column counts the partials from the block of row i+1 on
    if (lane == 0) pq.norms[lbi] = nrm;
  }
}

// a - v conj(wc) - w conj(vc)
template <typename R>
__device__ __forceinline__ cx<R> ht_rank2(cx<R> a, cx<R> v, cx<R> w, cx<R> vc, cx<R> wc) {
  a.re = fma(-w.im, vc.im, fma(-w.re, vc.re, fma(-v.im, wc.im, fma(-v.re, wc.re, a.re))));
  a.im = fma(w.re, vc.im, fma(-w.im, vc.re, fma(v.re, wc.im, fma(-v.im, wc.re, a.im))));
  return a;
}

// Entry kk of the accumulators (block kk / 4, register kk % 4) for a uniform
// kk: a tree of scalar branches (the empty asm keeps the compiler from merging
// its leaves to one indexed read, for which the array would go to memory).
template <int LO, int N, typename R, typename V>
__device__ __forceinline__ cx<R> ht_pick(const V (&re)[8], const V (&im)[8], int kk) {
  if constexpr (N == 1) {
    cx<R> t = cmk<R>(re[LO / 4][LO % 4], im[LO / 4][LO % 4]);
    asm("" : "+v"(t.re), "+v"(t.im));
    return t;
  } else {
    return kk < LO + N / 2 ? ht_pick<LO, N / 2, R>(re, im, kk) : ht_pick<LO + N / 2, N / 2, R>(re, im, kk);
  }
}

// Barrier that orders LDS only (__syncthreads also waits for the global stores in flight).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The last m <= HT_TAIL rows (columns ps .. n-1) of every matrix by one
// workgroup, the Hermitian block (both triangles) in registers in the layout
// of the matrix cores' accumulators, at the end of a 128 x 128 frame:
// wavefront w holds columns 16 w .. 16 w + 15 of all rows, lane (lrow, lk) the
// rows MfmaT::row(r, lk) of every 16-row block of column 16 w + lrow.  Per
// column j:
//   x = column j, read as the conjugate of row j (its update by column j-1
//     applied on the fly), shared; barrier;
//   A -= v w^H + w v^H of column j-1: the complex rank-2 update is one
//     four-deep real product each for the real and the imaginary part, one
//     matrix instruction per 16 x 16 block; beside it the scalars and
//     y_c = sum_r conj(a_rc) x_r, whole in the wavefront of its column; y and
//     row j+1 (for u = scale (y - beta a_{j+1}): v = scale x but for v_{j+1} =
//     1) shared; barrier;
//   g = v^H u and w = tau u - (|tau|^2 g / 2) v by every wavefront for itself,
//     v and w into its own operand copy P in LDS.
// Blocks of finished rows and wavefronts of finished columns drop out; rows
// above them are multiplied by zeros of v, w and x.
// Bound: the chain of m columns, of which the code takes what it can off the
// path between the barriers.  Order 82: 254 us with the block in LDS (three
// barriers, at most 92 rows), 195 with rows on lanes, columns in registers and
// operands broadcast from LDS, 167 now.  The two launches of a longer
// matrix cost 10 us a column.
template <typename R>
__global__ void __launch_bounds__(TAIL_THREADS) ht_tail(const HtProb<R> *pr) {
  typedef cx<R> C;
  typedef MfmaT<R> MF;
  typedef typename MF::v4 v4;
  static_assert(TAIL_THREADS == 512 && HT_TAIL == 128, "one wavefront per 16 columns");
  __shared__ C xs[HT_TAIL], us[HT_TAIL], as[HT_TAIL];
  __shared__ R P[8][HT_TAIL][4];                    // per wavefront: Re v, Im v, Re w, Im w of a row
  const HtProb<R> &q = pr[blockIdx.z];
  const int64_t n = q.n, lda = q.lda;
  if (n <= 0) return;
  const int64_t ps = ht_tail_start(n);
  const int o = HT_TAIL - (int)(n - ps);            // frame row of the first one
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 15, lk = lane >> 4, col = 16 * wave + lrow;
  MMF_GLOBAL C *A = (MMF_GLOBAL C *)q.A + ps + ps * lda;
  MMF_GLOBAL double *d = (MMF_GLOBAL double *)q.d + ps, *e = (MMF_GLOBAL double *)q.e + ps;
  MMF_GLOBAL C *tq = (MMF_GLOBAL C *)q.tau + ps;
  // register and lane group of row j
  constexpr bool PACKED = sizeof(R) == 4;           // MfmaT::row(r, lk) = 4 lk + r, else 4 r + lk
  const auto reg_of = [](int j) { return (j & ~15) / 4 + (PACKED ? j & 3 : (j >> 2) & 3); };
  const auto grp_of = [](int j) { return PACKED ? (j >> 2) & 3 : j & 3; };
  v4 are[8], aim[8];
#pragma unroll
  for (int b = 0; b < 8; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * b + MF::row(r, lk);
      const bool ok = row >= o && col >= o;
      const C t = gload(A + (ok ? (row >= col ? (row - o) + (col - o) * lda : (col - o) + (row - o) * lda) : 0));
      are[b][r] = t.re;
      aim[b][r] = t.im;
    }
  {                                                 // masks afresh: those of the addresses would not fit the scalar registers
    int c2 = col >= o ? col : -1;
    asm("" : "+v"(c2));
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * b + MF::row(r, lk);
        const bool ok = row >= o && c2 >= 0;
        are[b][r] = ok ? are[b][r] : R(0);
        aim[b][r] = !ok || row == c2 ? R(0) : row > c2 ? aim[b][r] : -aim[b][r];
      }
  }
#pragma unroll
  for (int t = 0; t < HT_TAIL * 4 / 64; ++t) P[wave][0][lane + 64 * t] = R(0);
  if (tid < HT_TAIL && tid < o) xs[tid] = cmk<R>(0, 0);
  C nx = ht_pick<0, 32, R>(are, aim, reg_of(o));    // row j of A (in lane group grp_of(j)) without the last update
  C vc = cmk<R>(0, 0), wc = vc, wj = vc;            // v, w of this lane's column, w of row j (v is 1 there)
  R vj = 0;
  C xa, xb, xc, tau, scale;                         // x of rows lane, 64 + lane and this lane's column
  R beta, yr, yi;
  for (int j = o;; ++j) {
    if (16 * wave + 15 >= j) {
      const C a = ht_rank2<R>(nx, cmk<R>(vj, 0), wj, vc, wc);
      if (lk == grp_of(j)) {
        xs[col] = cmk<R>(col > j ? a.re : R(0), col > j ? -a.im : R(0));
        if (col == j) d[j - o] = (double)a.re;
      }
    }
    if (j == HT_TAIL - 1) break;
    lds_barrier();
    const bool live = 16 * wave + 15 > j;
    if (live) {
      const R bre = -P[wave][col][lk ^ 2], bi = P[wave][col][lk ^ 3], bim = (lk & 1) ? -bi : bi;
      R pa[8];
#pragma unroll
      for (int b = 0; b < 8; ++b) pa[b] = P[wave][16 * b + lrow][lk];
      const C alpha = xs[j + 1];
      xa = xs[lane];
      xb = xs[64 + lane];
      xc = xs[col];
#pragma unroll
      for (int h = 0; h < 4; ++h)
        if (32 * h + 31 > j) {
#pragma unroll
          for (int b = 2 * h; b < 2 * h + 2; ++b) {
            are[b] = MF::run(pa[b], bre, are[b]);
            aim[b] = MF::run(pa[b], bim, aim[b]);
          }
        }
      const R xn = (lane == j + 1 ? R(0) : cabs2(xa)) + (64 + lane == j + 1 ? R(0) : cabs2(xb));
      ht_scalars<R>(alpha, wave_sum(xn), beta, tau, scale);
      R sr[4], si[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) sr[r] = si[r] = R(0);
#pragma unroll
      for (int h = 0; h < 4; ++h)
        if (32 * h + 31 > j) {
#pragma unroll
          for (int b = 2 * h; b < 2 * h + 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const C x = xs[16 * b + MF::row(r, lk)];
              sr[r] = fma(aim[b][r], x.im, fma(are[b][r], x.re, sr[r]));
              si[r] = fma(-aim[b][r], x.re, fma(are[b][r], x.im, si[r]));
            }
        }
      yr = rows_sum((sr[0] + sr[1]) + (sr[2] + sr[3]));
      yi = rows_sum((si[0] + si[1]) + (si[2] + si[3]));
      nx = ht_pick<0, 32, R>(are, aim, reg_of(j + 1));
      if (lk == grp_of(j + 1)) {
        us[col] = cmk<R>(yr, yi);
        as[col] = cconj(nx);
      }
    }
    lds_barrier();
    if (live) {
      const auto u_of = [&](C y, C a, bool on) {
        const C u = cmul(scale, cmk<R>(fma(-beta, a.re, y.re), fma(-beta, a.im, y.im)));
        return cmk<R>(on ? u.re : R(0), on ? u.im : R(0));
      };
      const bool ina = lane > j, inb = 64 + lane > j;
      const C ua = u_of(us[lane], as[lane], ina), ub = u_of(us[64 + lane], as[64 + lane], inb);
      const C uj = u_of(us[j + 1], as[j + 1], true), uc = u_of(cmk<R>(yr, yi), cconj(nx), col > j);
      C va = cmul(scale, xa), vb = cmul(scale, xb);
      if (lane == j + 1) va = cmk<R>(1, 0);
      if (64 + lane == j + 1) vb = cmk<R>(1, 0);
      vc = cmul(scale, xc);
      if (col == j + 1) vc = cmk<R>(1, 0);
      const R g = wave_sum(cmulc(va, ua).re + cmulc(vb, ub).re);
      const R hh = R(-0.5) * cabs2(tau) * g;
      wc = cadd(cmul(tau, uc), cscale(vc, hh));
      wj = cmul(tau, uj);
      wj.re += hh;
      vj = 1;
      const C wa = cadd(cmul(tau, ua), cscale(va, hh)), wb = cadd(cmul(tau, ub), cscale(vb, hh));
      R *p = P[wave][lane];
      p[0] = va.re; p[1] = va.im; p[2] = wa.re; p[3] = wa.im;
      p = P[wave][64 + lane];
      p[0] = vb.re; p[1] = vb.im; p[2] = wb.re; p[3] = wb.im;
      if (wave == 7) {                              // live to the end
        if (ina) A[lane - o + (j - o) * lda] = va;
        if (inb) A[64 + lane - o + (j - o) * lda] = vb;
        if (lane == 0) {
          e[j - o] = (double)beta;
          tq[j - o] = tau;
        }
      }
    }
  }
}

// Trailing update A[q0:, q0:] -= [V W] [W V]^H (lower tiles) after the panel
// starting at column p, for every matrix of the table.
template <typename R>
__global__ void __launch_bounds__(GEMM_THREADS, 2) ht_her2k(const HtProb<R> *pr, int64_t p) {
  __shared__ R lds[GEMM_LDS_ELEMS];
  const HtProb<R> &q = pr[blockIdx.z];
  const int64_t n = q.n;
  if (p >= ht_tail_start(n)) return;
  const int64_t q0 = p + HT_NB;
  const int64_t M = n - q0;
  const int64_t m0 = (int64_t)blockIdx.x * GT_M, n0 = (int64_t)blockIdx.y * GT_N;
  if (m0 >= M || n0 >= M || m0 + GT_M <= n0) return;
  GemmArgs g = gemm_args(M, M, 2 * HT_NB, q.P3 + q0, n, q.P3 + q0 + (int64_t)HT_NB * n, n,
                         q.A + q0 + q0 * q.lda, q.lda, -1.0, 0.0, 1.0, 0.0);
  g.lower = 1;
  gemm_tile_t<R, true, A_N, B_C>(g, m0, n0, lds);
}

// ---------------------------------------------------------------- host
// Grouped reduction of `count` matrices described by the device table pr
// (orders nh[0..count) on the host).
template <typename R>
int hetrd_grouped(const HtProb<R> *pr, const int64_t *nh, int64_t count, hipStream_t st) {
  int64_t nmax = 0;
  for (int64_t c = 0; c < count; ++c) nmax = nh[c] > nmax ? nh[c] : nmax;
  if (nmax <= 0 || count <= 0) return MMF_OK;
  const unsigned Z = (unsigned)count;
  const int64_t ps = ht_tail_start(nmax);
  for (int64_t p = 0; p < ps; p += HT_NB) {
    int rows = 0, strip = 1;                         // most strip rows and longest strip of any matrix in this panel
    for (int64_t c = 0; c < count; ++c) {
      if (p >= ht_tail_start(nh[c])) continue;
      const int ch = ht_strip(nh[c], p), sl = ht_strips(nh[c], p, ch, 0) + 1;   // two folded columns have at most these
      strip = ch > strip ? ch : strip;
      rows = sl > rows ? sl : rows;
    }
    hipLaunchKernelGGL(ht_colnorm<R>, dim3(cdiv(cdiv(nmax, HV_T) - p / HV_T, 4), 1, Z), dim3(256), 0, st, pr, p);
    MMF_LAUNCH_CHECK();
    for (int k = 0; k < HT_NB; ++k) {
      const int64_t i = p + k;
      // anchored 64-blocks of the largest matrix: block columns b0 .. nb-1
      const int64_t nbl = (nmax + HV_T - 1) / HV_T - (i + 1) / HV_T;
      const int64_t gx = (nbl + 1) / 2;
      int64_t items = 0;                             // most diagonal, edge and product workgroups of any matrix
      for (int64_t c = 0; c < count; ++c) {
        if (p >= ht_tail_start(nh[c])) continue;
        const int64_t dr = ht_dot_rows(nh[c]), nb = (nh[c] + HV_T - 1) / HV_T - (i + 1) / HV_T;
        const int64_t it = 2 * nb + (2 * k + 3) / 4 * ((nh[c] - i - 1 + dr - 1) / dr);   // four products per workgroup
        items = it > items ? it : items;
      }
      const int ks = ktimer_begin(sizeof(R) == 8 ? "hemv" : "hemv_c64", st);
      const dim3 grid((unsigned)gx, (unsigned)(rows + (items + gx - 1) / gx), Z);
      if ((int64_t)sizeof(cx<R>) * (nmax - p) * (nmax - p) / 2 > HV_NT_BYTES)
        hipLaunchKernelGGL((ht_column<R, true, true>), grid, dim3(256), 0, st, pr, p, k, rows);
      else if (strip > 1)
        hipLaunchKernelGGL((ht_column<R, false, true>), grid, dim3(256), 0, st, pr, p, k, rows);
      else
        hipLaunchKernelGGL((ht_column<R, false, false>), grid, dim3(256), 0, st, pr, p, k, rows);
      MMF_LAUNCH_CHECK();
      if (ks >= 0) {
        // algorithmic bytes: the lower triangle of every trailing matrix, read
        // once, plus the 2k panel columns and v read by the fused dot products
        double bytes = 0.0;
        for (int64_t c = 0; c < count; ++c) {
          const double mc = i < ht_tail_start(nh[c]) ? (double)(nh[c] - i - 1) : 0.0;
          if (mc > 0) bytes += 2.0 * sizeof(R) * (mc * (mc + 1.0) / 2.0 + (k > 0 ? (2.0 * k + 1.0) * mc : 0.0));
        }
        ktimer_end(ks, st, bytes);
      }
      if (nbl * count <= HF_WIDE_MAX)
        hipLaunchKernelGGL((ht_finish<R, true>), dim3((unsigned)nbl, 1, Z), dim3(512), 0, st, pr, p, k);
      else
        hipLaunchKernelGGL((ht_finish<R, false>), dim3((unsigned)nbl, 1, Z), dim3(256), 0, st, pr, p, k);
      MMF_LAUNCH_CHECK();
    }
    const unsigned t = cdiv(nmax - p - HT_NB, GT_M);
    hipLaunchKernelGGL(ht_her2k<R>, dim3(t, t, Z), dim3(GEMM_THREADS), 0, st, pr, p);
    MMF_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(ht_tail<R>, dim3(1, 1, Z), dim3(TAIL_THREADS), 0, st, pr);
  MMF_LAUNCH_CHECK();
  return MMF_OK;
}

// bytes of the one-entry table placed in front of a single reduction's workspace
constexpr size_t HT_TABLE_BYTES = 256;

template <typename R>
int hetrd_run_t(int64_t n, cx<R> *A, int64_t lda, double *d, double *e, cx<R> *tau, void *work,
                size_t bytes, hipStream_t st) {
  if (n <= 0) return MMF_OK;
  static_assert(sizeof(HtProb<R>) <= HT_TABLE_BYTES, "table entry");
  HtWs<R> w = hetrd_ws<R>(n, (char *)work + HT_TABLE_BYTES);
  if (bytes < w.bytes + HT_TABLE_BYTES) return MMF_ERR_WORKSPACE;
  HtProb<R> *pr = reinterpret_cast<HtProb<R> *>(work);
  const HtProb<R> q = ht_prob<R>(n, A, lda, d, e, tau, w);
  int rc = table_write(pr, &q, 1, st);
  if (rc) return rc;
  return hetrd_grouped<R>(pr, &n, 1, st);
}

// Batch: entry c reduces A[c] (order n[c] >= 1) using the stage workspace
// stage[c] (laid out as for a single reduction); the problem table goes to
// `table` (count * STAGE_TABLE_BYTES device bytes).
template <typename R>
int hetrd_batched_t(int64_t count, const int64_t *n, cx<R> *const *A, const int64_t *lda, double *const *d,
                    double *const *e, cx<R> *const *tau, void *const *stage, void *table, hipStream_t st) {
  static_assert(sizeof(HtProb<R>) <= STAGE_TABLE_BYTES, "table entry");
  std::vector<HtProb<R>> h((size_t)count);
  for (int64_t c = 0; c < count; ++c)
    h[c] = ht_prob<R>(n[c], A[c], lda[c], d[c], e[c], tau[c],
                      hetrd_ws<R>(n[c], (char *)stage[c] + HT_TABLE_BYTES));
  HtProb<R> *pr = reinterpret_cast<HtProb<R> *>(table);
  const int rc = table_write(pr, h.data(), count, st);
  if (rc) return rc;
  return hetrd_grouped<R>(pr, n, count, st);
}

int hetrd_batched(int64_t count, const int64_t *n, mmf_z *const *A, const int64_t *lda, double *const *d,
                  double *const *e, mmf_z *const *tau, void *const *stage, void *table, hipStream_t st) {
  return hetrd_batched_t<double>(count, n, reinterpret_cast<cd *const *>(A), lda, d, e,
                                 reinterpret_cast<cd *const *>(tau), stage, table, st);
}

int hetrd_batched_c64(int64_t count, const int64_t *n, void *const *A, const int64_t *lda, double *const *d,
                      double *const *e, void *const *tau, void *const *stage, void *table, hipStream_t st) {
  return hetrd_batched_t<float>(count, n, reinterpret_cast<cf *const *>(A), lda, d, e,
                                reinterpret_cast<cf *const *>(tau), stage, table, st);
}

int hetrd_run(int64_t n, mmf_z *A, int64_t lda, double *d, double *e, mmf_z *tau, void *work,
              size_t bytes, hipStream_t st) {
  return hetrd_run_t<double>(n, reinterpret_cast<cd *>(A), lda, d, e, reinterpret_cast<cd *>(tau), work,
                             bytes, st);
}

size_t hetrd_ws_bytes_c64(int64_t n) { return hetrd_ws_bytes_t<float>(n) + 256; }
int hetrd_run_c64(int64_t n, void *A, int64_t lda, double *d, double *e, void *tau, void *work,
                  size_t bytes, hipStream_t st) {
  return hetrd_run_t<float>(n, reinterpret_cast<cf *>(A), lda, d, e, reinterpret_cast<cf *>(tau), work,
                            bytes, st);
}

}  // namespace mmf

using namespace mmf;

extern "C" int mmf_hetrd(int64_t n, mmf_z *A, int64_t lda, double *d, double *e, mmf_z *tau,
                         void *work, size_t work_bytes, void *stream) {
  if (n < 0) return -1;
  if (!A) return -2;
  if (lda < n || lda < 1) return -3;
  if (!d) return -4;
  if (n > 1 && !e) return -5;
  if (n > 1 && !tau) return -6;
  if (!work) return -7;
  if (work_bytes < hetrd_ws_bytes(n)) return -8;
  return hetrd_run(n, A, lda, d, e, tau, work, work_bytes, (hipStream_t)stream);
}
