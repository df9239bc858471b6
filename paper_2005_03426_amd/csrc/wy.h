// Triangular factor of 64 Householder reflectors in compact-WY form (internal).
#pragma once
#include "common.h"

namespace mmf {

constexpr int WY_N = 64, WY_LD = 65, WY_THREADS = 256;

// T[r][c] of the array W below
template <typename R>
__device__ inline cx<R> wy_t(const cx<R> (*W)[WY_LD], int r, int c) {
  return r <= c ? W[c][r] : cmk<R>(0, 0);
}
// The joins of neighbouring L x L pieces: X = G_12 T_2, kept where T_12 will be,
// then T_12 = -T_1 X.
template <typename R, int L>
__device__ inline void wy_join(cx<R> (*W)[WY_LD]) {
  constexpr int PER = 32 * L / WY_THREADS;          // entries of a thread
  const int tid = threadIdx.x;
  cx<R> t[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int e = tid + WY_THREADS * m, i = e % L, c = (e / L) % L, o1 = 2 * L * (e / (L * L)), o2 = o1 + L;
    cx<R> s = cmk<R>(0, 0);
#pragma unroll 8
    for (int k = 0; k < L; ++k) s = cadd(s, cmul(W[o1 + i][o2 + k], wy_t<R>(W, o2 + k, o2 + c)));
    W[o2 + c][o1 + i] = s;
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int e = tid + WY_THREADS * m, i = e % L, c = (e / L) % L, o1 = 2 * L * (e / (L * L)), o2 = o1 + L;
    t[m] = cmk<R>(0, 0);
#pragma unroll 8
    for (int k = 0; k < L; ++k) t[m] = cadd(t[m], cmul(wy_t<R>(W, o1 + i, o1 + k), W[o2 + c][o1 + k]));
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int e = tid + WY_THREADS * m, i = e % L, c = (e / L) % L, o1 = 2 * L * (e / (L * L)), o2 = o1 + L;
    W[o2 + c][o1 + i] = cmk<R>(-t[m].re, -t[m].im);
  }
  __syncthreads();
}

// H_0 H_1 ... H_63 = I - V T V^H from the Gram matrix G = V^H V and tau (LDS):
// T[k][k] = tau_k, T[0:k, k] = -tau_k T[0:k, 0:k] G[0:k, k]; a zero tau leaves
// a zero row and column.  One array W (LDS) holds both: on entry G[j][k], j < k,
// at W[j][k], on return also T[r][c], r <= c, at W[c][r] (wy_t reads T with its
// zeros).  Two arrays of 133 KB together had to wait until both workgroups of
// the band reduction's update (66.6 KB each) had left a CU: 118 us a panel at
// order 20808, up to 1073, against 31, up to 71, in one array.
// The recurrence is a chain of one step per reflector, so it runs on 16 x 16
// diagonal blocks only, one wavefront each (lane = row, the row in registers),
// and the blocks are joined 16 + 16, then 32 + 32, by T_12 = -T_1 G_12 T_2 with
// all 256 threads.  On a CU of its own the 64-step recurrence took 147 us in one
// wavefront and 62 us in four; with two arrays this form took 29 and 23 in the
// two kernels that call it.
// Called by the whole workgroup of WY_THREADS; W and tau complete before.
template <typename R>
__device__ inline void wy_tfactor(cx<R> (*W)[WY_LD], const cx<R> *tau) {
  const int tid = threadIdx.x;
  {
    const int o = 16 * (tid >> 6), r = tid & 15;
    cx<R> t[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const cx<R> tk = tau[o + k];
      cx<R> s = cmk<R>(0, 0);
#pragma unroll
      for (int j = 0; j < k; ++j) s = cadd(s, cmul(t[j], W[o + j][o + k]));
      const cx<R> u = cmul(tk, s);
      t[k] = r < k ? cmk<R>(-u.re, -u.im) : (r == k ? tk : cmk<R>(0, 0));
    }
    if ((tid & 63) < 16) {
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (r <= k) W[o + k][o + r] = t[k];
    }
  }
  __syncthreads();
  wy_join<R, 16>(W);
  wy_join<R, 32>(W);
}

}  // namespace mmf
