// Triangular factor of 64 Householder reflectors in compact-WY form (internal).
#pragma once
#include "common.h"

namespace mmf {

constexpr int WY_N = 64, WY_LD = 65, WY_THREADS = 256;

// H_0 H_1 ... H_63 = I - V T V^H from the Gram matrix G = V^H V (upper part,
// G[j][k], in LDS) and tau (LDS): T[k][k] = tau_k,
// T[0:k, k] = -tau_k T[0:k, 0:k] G[0:k, k], zero below the diagonal; a zero
// tau leaves a zero row and column.  The recurrence is a chain of one step per
// reflector, so it runs on 16 x 16 diagonal blocks only, one wavefront each
// (lane = row, the row in registers), and the blocks are joined 16 + 16, then
// 32 + 32, by T_12 = -T_1 G_12 T_2 with all 256 threads.  The 64-step
// recurrence took 147 us in one wavefront and 62 us in four, this form 29 and
// 23 in the two kernels that call it.
// Called by the whole workgroup of WY_THREADS; G and tau complete before.
template <typename R>
__device__ inline void wy_tfactor(const cx<R> (*G)[WY_LD], cx<R> (*T)[WY_LD], const cx<R> *tau) {
  const int tid = threadIdx.x;
  {
    const int o = 16 * (tid >> 6), r = tid & 15;
    cx<R> t[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const cx<R> tk = tau[o + k];
      cx<R> s = cmk<R>(0, 0);
#pragma unroll
      for (int j = 0; j < k; ++j) s = cadd(s, cmul(t[j], G[o + j][o + k]));
      const cx<R> u = cmul(tk, s);
      t[k] = r < k ? cmk<R>(-u.re, -u.im) : (r == k ? tk : cmk<R>(0, 0));
    }
    if ((tid & 63) < 16) {
#pragma unroll
      for (int k = 0; k < 16; ++k) T[o + r][o + k] = t[k];
    }
    for (int e = tid; e < WY_N * WY_N; e += WY_THREADS) {
      const int i = e & 63, c = e >> 6;
      if ((i >> 4) != (c >> 4)) T[i][c] = cmk<R>(0, 0);
    }
  }
  __syncthreads();
  for (int L = 16; L < WY_N; L *= 2) {
    // X = G_12 T_2, kept in the still empty lower-left piece of the pair
    for (int e = tid; e < 32 * L; e += WY_THREADS) {
      const int i = e % L, c = (e / L) % L, o1 = 2 * L * (e / (L * L)), o2 = o1 + L;
      cx<R> s = cmk<R>(0, 0);
#pragma unroll 8
      for (int k = 0; k < L; ++k) s = cadd(s, cmul(G[o1 + i][o2 + k], T[o2 + k][o2 + c]));
      T[o2 + i][o1 + c] = s;
    }
    __syncthreads();
    for (int e = tid; e < 32 * L; e += WY_THREADS) {
      const int i = e % L, c = (e / L) % L, o1 = 2 * L * (e / (L * L)), o2 = o1 + L;
      cx<R> s = cmk<R>(0, 0);
#pragma unroll 8
      for (int k = 0; k < L; ++k) s = cadd(s, cmul(T[o1 + i][o1 + k], T[o2 + k][o1 + c]));
      T[o1 + i][o2 + c] = cmk<R>(-s.re, -s.im);
    }
    __syncthreads();
    for (int e = tid; e < 32 * L; e += WY_THREADS) {
      const int i = e % L, c = (e / L) % L, o1 = 2 * L * (e / (L * L)), o2 = o1 + L;
      T[o2 + i][o1 + c] = cmk<R>(0, 0);
    }
    __syncthreads();
  }
}

}  // namespace mmf
