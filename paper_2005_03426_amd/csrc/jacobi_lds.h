// Hermitian eigensolver for one small matrix held in LDS by one workgroup
// (internal header): two-sided cyclic Jacobi with the parallel round-robin
// ordering of Brent and Luk (SIAM J. Sci. Stat. Comput. 6, 1985), each step
// rotating n/2 disjoint index pairs at once.  A rotation first removes the
// phase of t_pq with a diagonal unitary, then applies the real symmetric
// Jacobi rotation that zeroes the now-real 2 x 2 off-diagonal (the classical
// choice of the smaller rotation angle, Golub and Van Loan Sec. 8.5).
#pragma once
#include "common.h"

namespace mmf {

constexpr int JAC_NMAX = 64;            // largest order (T and Q: 2 x 64 x 65 complex = 130 KiB of LDS)
constexpr int JAC_LD = JAC_NMAX + 1;    // row stride of T and Q for the largest order
// |tpq|^2 below which the entry is scaled to about one before it is squared: a
// subnormal square keeps only a few bits, the phase tpq / |tpq| formed from it
// is not of modulus one and the rotation not unitary.  The fill-in of a weakly
// driven ladder (couplings V far from the diagonal as V^k) comes through that
// range: at V = 1e-5, order 50, Q^H Q was off by 0.25.
constexpr double JAC_SCALE = 1e-280;

// LDS of one solve: T and Q (n x n, row r at r * ld, ld >= n + 1 against bank
// conflicts), the rotations of one step and a reduction scratch.
struct JacView {
  cd *T, *Q;
  int ld;
  double (*rot)[4];                     // per pair: c, s, Re ph, Im ph
  int (*pair)[2];                       // per pair: p < q
  double (*red)[16];                    // [2][16]
};

// Bytes of LDS a JacView of order n takes (laid out by jac_view).
__host__ __device__ constexpr size_t jac_lds_bytes(int n) {
  return 2 * (size_t)n * (size_t)(n + 1) * sizeof(cd) + (size_t)(n / 2 + 1) * (4 * sizeof(double) + 2 * sizeof(int)) +
         32 * sizeof(double) + 64;
}

__device__ inline JacView jac_view(char *lds, int nmax) {
  JacView v;
  v.ld = nmax + 1;
  v.T = reinterpret_cast<cd *>(lds);
  v.Q = v.T + (size_t)nmax * v.ld;
  v.rot = reinterpret_cast<double (*)[4]>(v.Q + (size_t)nmax * v.ld);
  v.red = reinterpret_cast<double (*)[16]>(&v.rot[nmax / 2 + 1][0]);
  v.pair = reinterpret_cast<int (*)[2]>(&v.red[2][0]);
  return v;
}

// Position j of the round-robin schedule at step r < m - 1 for m players (m
// even): player 0 stays, the others rotate.
__device__ inline int jac_player(int j, int r, int m) {
  const int x = j - 1 + r;
  return j == 0 ? 0 : (x >= m - 1 ? x - (m - 1) : x) + 1;
}

// Sum over the workgroup of two doubles (result valid in every thread).
template <int NT>
__device__ inline void jac_sum2(const JacView &L, double &a, double &b) {
  a = wave_sum(a);
  b = wave_sum(b);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { L.red[0][w] = a; L.red[1][w] = b; }
  __syncthreads();
  a = 0.0;
  b = 0.0;
#pragma unroll
  for (int q = 0; q < NT / 64; ++q) { a += L.red[0][q]; b += L.red[1][q]; }
}

// Diagonalises the Hermitian n x n matrix in L.T (n <= JAC_NMAX) and
// accumulates the rotations into L.Q (which the caller initialises, e.g. to
// the identity): on return the eigenvalues are on the diagonal of T
// (unsorted) and the eigenvectors in the columns of Q.  Sweeps until the
// off-diagonal Frobenius norm is below 1e-16 of the total, at most max_sweeps
// of them; returns whether it ended below (n eps)^2 of the total in squares
// (eigenvalues then within about n eps ||T||).  Every thread of the NT-thread
// workgroup calls it.
//
// A step is a chain: the rotations from T, then T and Q by the rotations, two
// barriers.  Thread (a, b) = (tid / np, tid % np) keeps the rotation of pair b
// and owns the 2 x 2 blocks of T at pairs (a, b), (a + rows, b), ..., which it
// rotates from both sides at once, so T is read and written once per step and
// no block is touched by two threads; Q takes its column rotations in the same
// phase.  Rotating columns, then rows
// (four barriers, an integer division per element, square roots and divisions
// in the angles) took 545 us for 512 matrices of order 34 with 256 threads,
// this form 336.  (Groups of a power of two lanes: 456; two blocks or four rows
// in flight per thread: 373, with 144 registers against 98; rotations formed
// by every wavefront for itself and read per block: 473.)
template <int NT>
__device__ bool jacobi_herm_lds(const JacView &L, int n, int max_sweeps) {
  const int tid = threadIdx.x;
  const int ld = L.ld;
  const int m = n + (n & 1);            // players; an odd n gets a dummy index n (skipped)
  const int np = m / 2;
  const int rows = NT / np, a0 = tid / np, b0 = a0 < rows ? tid - a0 * np : np;   // the last NT % np threads idle
  double off = 0.0, tot = 0.0;
  __syncthreads();
  for (int sweep = 0;; ++sweep) {
    off = 0.0;
    tot = 0.0;
    for (int r = a0; b0 < np && r < n; r += rows)
      for (int c = b0; c < n; c += np) {
        const double v = cabs2(L.T[r * ld + c]);
        tot += v;
        if (r != c) off += v;
      }
    jac_sum2<NT>(L, off, tot);
    if (off <= 1e-32 * tot || off == 0.0 || sweep == max_sweeps) break;
    for (int step = 0; step < m - 1; ++step) {
      // rotation of every pair of this step
      if (tid < np) {
        int p = jac_player(tid, step, m), q = jac_player(m - 1 - tid, step, m);
        if (p > q) { const int t = p; p = q; q = t; }
        double cs = 1.0, sn = 0.0, phr = 1.0, phi = 0.0;
        if (q < n) {
          cd tpq = L.T[p * ld + q];
          double gap = L.T[q * ld + q].re - L.T[p * ld + p].re, r2 = cabs2(tpq);
          if (r2 < JAC_SCALE) {             // the angles depend on gap / |tpq| and tpq / |tpq| alone
            int ex;
            (void)frexp(fmax(fabs(tpq.re), fabs(tpq.im)), &ex);
            tpq = cmake(ldexp(tpq.re, -ex), ldexp(tpq.im, -ex));
            gap = ldexp(gap, -ex);
            r2 = cabs2(tpq);
          }
          if (r2 > 0.0) {
            const double ri = rsqrt(r2);
            phr = tpq.re * ri;
            phi = tpq.im * ri;
            const double theta = 0.5 * gap * ri;
            const double t = copysign(1.0 / (fabs(theta) + sqrt(fma(theta, theta, 1.0))), theta);
            cs = rsqrt(fma(t, t, 1.0));
            sn = t * cs;
          }
        }
        L.pair[tid][0] = p;
        L.pair[tid][1] = q;
        L.rot[tid][0] = cs;
        L.rot[tid][1] = sn;
        L.rot[tid][2] = phr;
        L.rot[tid][3] = phi;
      }
      __syncthreads();
      if (b0 < np) {
        // pair of this lane: J = [[c, s], [-s conj(ph), c conj(ph)]] on its columns (pb, qb)
        const int pb = L.pair[b0][0], qb = L.pair[b0][1];
        const bool wb = qb < n;                   // the dummy's partner keeps its column
        const double cb = L.rot[b0][0], sb = L.rot[b0][1];
        const cd phb = cmake(L.rot[b0][2], -L.rot[b0][3]);
        const cd j10 = cscale(phb, -sb), j11 = cscale(phb, cb);
        // T <- J^H T J: block (a, b)
        for (int a = a0; a < np; a += rows) {
          const int pa = L.pair[a][0], qa = L.pair[a][1];
          const bool wa = qa < n;
          const double ca = L.rot[a][0], sa = L.rot[a][1];
          const cd pha = cmake(L.rot[a][2], L.rot[a][3]);
          cd pp = L.T[pa * ld + pb], pq = wb ? L.T[pa * ld + qb] : cmake(0.0, 0.0);
          cd qp = wa ? L.T[qa * ld + pb] : cmake(0.0, 0.0), qq = wa && wb ? L.T[qa * ld + qb] : cmake(0.0, 0.0);
          const cd xpp = cadd(cscale(pp, cb), cmul(pq, j10)), xpq = cadd(cscale(pp, sb), cmul(pq, j11));
          const cd xqp = cadd(cscale(qp, cb), cmul(qq, j10)), xqq = cadd(cscale(qp, sb), cmul(qq, j11));
          const cd s0 = cscale(pha, sa), c0 = cscale(pha, ca);
          pp = csub(cscale(xpp, ca), cmul(s0, xqp));
          pq = csub(cscale(xpq, ca), cmul(s0, xqq));
          qp = cadd(cscale(xpp, sa), cmul(c0, xqp));
          qq = cadd(cscale(xpq, sa), cmul(c0, xqq));
          if (a == b0) {                          // the rotated pair itself: diagonal
            pq = qp = cmake(0.0, 0.0);
            pp.im = qq.im = 0.0;
          }
          L.T[pa * ld + pb] = pp;
          if (wb) L.T[pa * ld + qb] = pq;
          if (wa) L.T[qa * ld + pb] = qp;
          if (wa && wb) L.T[qa * ld + qb] = qq;
        }
        // Q <- Q J
        if (wb)
          for (int k = a0; k < n; k += rows) {
            const cd qp = L.Q[k * ld + pb], qq = L.Q[k * ld + qb];
            L.Q[k * ld + pb] = cadd(cscale(qp, cb), cmul(qq, j10));
            L.Q[k * ld + qb] = cadd(cscale(qp, sb), cmul(qq, j11));
          }
      }
      __syncthreads();
    }
  }
  const double tol = (double)n * 2.220446049250313e-16;
  return off <= tol * tol * tot;
}

}  // namespace mmf
