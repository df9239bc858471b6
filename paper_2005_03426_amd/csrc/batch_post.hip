// Batched assembly and observables of many small Floquet problems (a
// parameter sweep): H_F of every problem in one launch, and U(t, t0) (Eqs.
// 3-5) with the averaged transition probabilities of every problem in a fixed
// handful of launches, whatever the batch size -- instead of several launches
// per problem.  Each kernel reads its problem from a device table (BEnt).
//
// U_ij(t_q, t0) = sum_a e^{-i eps_a (t_q - t0)} [sum_s e^{+i n_s.w t_q} Phi[i + D s, a]] conj(Phi[j + D s0, a]):
//   ob_phases  B[s][q] = e^{+i n_s.w t_q}
//   ob_project Y[q][a][i] = e^{-i eps_a (t_q - t0)} sum_s B[s][q] Phi[i + D s, a]   (one column a per step)
//   ob_contract U[q](i, j) = sum_a Y[q][a][i] conj(Phi[j + D s0, a])              (fixed order)
// P[i, j] = sum_a (sum_n |Phi[(i,n),a]|^2) |Phi[(j,0),a]|^2, with the
// degenerate-pair check of mmf_avg_prob, by per-problem partials and a sum.
// Everything in FP64 on the vector units: the per-problem products are far
// too small for the matrix cores.
#include <algorithm>
#include <vector>
#include "common.h"
#include "problem.h"
#include "batch.h"
#include "table.h"

namespace mmf {

constexpr int OB_THREADS = 256;
constexpr int OB_PROJ_GRID = 1024;    // most workgroups per problem row of the projection (they loop over columns)
constexpr int AP_GROUPS = 64;         // averaged-probability partials per problem
constexpr double OB_CLUSTER_REL = 1e-8;
constexpr double OB_SHARED_WEIGHT = 1e-20;

__global__ void __launch_bounds__(OB_THREADS) ob_phases(const BEnt *__restrict__ tab) {
  const BEnt &b = tab[blockIdx.y];
  const int64_t e = (int64_t)blockIdx.x * OB_THREADS + threadIdx.x;
  if (e >= b.S * b.T) return;
  const int q = (int)(e % b.T);
  int64_t rem = e / b.T;
  double theta = 0.0;
  for (int l = 0; l < BMAX_F; ++l) {
    if (l >= b.F) break;
    const int64_t dig = rem % b.radix[l];
    rem /= b.radix[l];
    theta += (double)(b.N[l] - (int32_t)dig) * b.omega[l];
  }
  double sn, cs;
  sincos(theta * b.t[q], &sn, &cs);
  b.B[e] = cmake(cs, sn);
}

// Columns a of problem blockIdx.y.  With D T <= 128 a workgroup takes
// 256 / (D T) columns at a time (thread e = i + D q of a column), otherwise one
// column with up to eight outputs per thread; the columns' rows are staged in
// LDS in chunks of whole sites.  For 512 problems of order 34 (T = 32) a grid
// of 1024 workgroups per problem, one column and 64 busy threads each, took
// 289 us, mostly empty workgroups; now 34.
__host__ __device__ inline int ob_project_cols(int D, int T) { return D * T <= OB_THREADS / 2 ? OB_THREADS / (D * T) : 1; }

// KMAX: most outputs per thread over the batch (1 or 8).
template <int KMAX>
__global__ void __launch_bounds__(OB_THREADS) ob_project(const BEnt *__restrict__ tab) {
  __shared__ cd col[2048];
  const BEnt &b = tab[blockIdx.y];
  const int D = b.D, T = b.T, DT = D * T;
  const int tid = threadIdx.x;
  const int CB = ob_project_cols(D, T);
  const int lim = 2048 / CB, chunk = lim / D * D;     // rows of a column staged at a time
  const int cb = CB > 1 ? tid / DT : 0;
  for (int64_t a0 = (int64_t)blockIdx.x * CB; a0 < b.M; a0 += (int64_t)gridDim.x * CB) {
    const int nc = (int)(b.M - a0 < CB ? b.M - a0 : CB);
    double sn, cs;
    cd acc[KMAX];
    for (int k = 0; k < KMAX; ++k) acc[k] = cmake(0.0, 0.0);
    for (int64_t r0 = 0; r0 < b.M; r0 += chunk) {
      const int nr = (int)((b.M - r0 < chunk) ? b.M - r0 : chunk);
      __syncthreads();
      for (int c = 0; c < nc; ++c)
        for (int r = tid; r < nr; r += OB_THREADS) col[c * lim + r] = b.HF[(a0 + c) * b.ld + r0 + r];
      __syncthreads();
      const int64_t s_lo = r0 / D, s_hi = (r0 + nr) / D;      // r0 and nr are multiples of D (so is M)
      if (CB > 1) {
        const int e = tid - cb * DT, i = e % D, q = e / D;
        if (cb < nc) {
          cd s = acc[0];
          const cd *cc = col + cb * lim + i - r0;
#pragma unroll 4
          for (int64_t site = s_lo; site < s_hi; ++site) s = cadd(s, cmul(b.B[site * T + q], cc[D * site]));
          acc[0] = s;
        }
        continue;
      }
      for (int k = 0; k < KMAX; ++k) {
        const int e = tid + OB_THREADS * k;
        if (e >= DT) break;
        const int i = e % D, q = e / D;
        cd s = acc[k];
        for (int64_t site = s_lo; site < s_hi; ++site)
          s = cadd(s, cmul(b.B[site * T + q], col[i + D * site - r0]));
        acc[k] = s;
      }
    }
    if (CB > 1) {
      const int e = tid - cb * DT, i = e % D, q = e / D;
      if (cb < nc) {
        const int64_t a = a0 + cb;
        sincos(-(b.w[a] * (b.t[q] - b.t0)), &sn, &cs);
        b.Y[((int64_t)q * b.M + a) * D + i] = cmul(acc[0], cmake(cs, sn));
      }
      continue;
    }
    for (int k = 0; k < KMAX; ++k) {
      const int e = tid + OB_THREADS * k;
      if (e >= DT) break;
      const int i = e % D, q = e / D;
      sincos(-(b.w[a0] * (b.t[q] - b.t0)), &sn, &cs);
      b.Y[((int64_t)q * b.M + a0) * D + i] = cmul(acc[k], cmake(cs, sn));
    }
  }
}

// U of problem blockIdx.y.  With D^2 <= 64 a workgroup takes 64 / D^2 times,
// each with four groups of D^2 threads that share the columns (summed in group
// order); otherwise one time, up to 16 elements per thread.  The zero-site rows
// are staged in LDS.  512 problems of order 34 at 32 times: one time and four
// busy threads per workgroup took 133 us, this form 7.
constexpr int OB_PARTS = 4;
__host__ __device__ inline int ob_contract_times(int D) { return D * D <= 64 ? OB_THREADS / (OB_PARTS * D * D) : 1; }

// KMAX: most elements of U per thread over the batch (1 or 16).
template <int KMAX>
__global__ void __launch_bounds__(OB_THREADS) ob_contract(const BEnt *__restrict__ tab) {
  __shared__ cd ps[2048];
  __shared__ cd red[OB_THREADS];
  const BEnt &b = tab[blockIdx.y];
  const int D = b.D, DD = D * D;
  const int QB = ob_contract_times(D);
  const int q0 = blockIdx.x * QB;
  if (q0 >= b.T) return;
  const int tid = threadIdx.x;
  const int sub = 2048 / D;
  const bool small = DD <= 64;
  const int ql = small ? tid / (OB_PARTS * DD) : 0, rest = small ? tid - ql * OB_PARTS * DD : tid;
  const int g = small ? rest / DD : 0;
  const int q = q0 + ql;
  cd acc[KMAX];
  for (int k = 0; k < KMAX; ++k) acc[k] = cmake(0.0, 0.0);
  for (int64_t ab = 0; ab < b.M; ab += sub) {
    const int na = (int)((b.M - ab < sub) ? b.M - ab : sub);
    __syncthreads();
    for (int e = tid; e < na * D; e += OB_THREADS) {
      const int aa = e / D, i = e - aa * D;
      ps[e] = cconj(b.HF[i + (int64_t)D * b.s0 + (ab + aa) * b.ld]);
    }
    __syncthreads();
    if (small) {
      if (ql < QB && q < b.T) {
        const int e = rest - g * DD, i = e % D, j = e / D;
        const cd *y = b.Y + ((int64_t)q * b.M + ab) * D + i;
        cd s = acc[0];
#pragma unroll 4
        for (int aa = g; aa < na; aa += OB_PARTS) s = cadd(s, cmul(y[(int64_t)aa * D], ps[aa * D + j]));
        acc[0] = s;
      }
      continue;
    }
    for (int k = 0; k < KMAX; ++k) {
      const int e = tid + OB_THREADS * k;
      if (e >= DD) break;
      const int i = e % D, j = e / D;
      const cd *y = b.Y + ((int64_t)q * b.M + ab) * D + i;
      cd s = acc[k];
      for (int aa = 0; aa < na; ++aa) s = cadd(s, cmul(y[(int64_t)aa * D], ps[aa * D + j]));
      acc[k] = s;
    }
  }
  if (small) {
    red[tid] = acc[0];
    __syncthreads();
    if (ql < QB && q < b.T && g == 0) {
      cd s = red[tid];
      for (int gg = 1; gg < OB_PARTS; ++gg) s = cadd(s, red[tid + gg * DD]);
      b.U[(int64_t)q * DD + rest] = s;
    }
    return;
  }
  for (int k = 0; k < KMAX; ++k) {
    const int e = tid + OB_THREADS * k;
    if (e >= DD) break;
    b.U[(int64_t)q * DD + e] = acc[k];
  }
}

// Averaged-probability partials of problem blockIdx.y: group g = blockIdx.x
// takes the columns a = g, g + AP_GROUPS, ...
__global__ void __launch_bounds__(OB_THREADS) ob_avgprob(const BEnt *__restrict__ tab) {
  __shared__ double red[OB_THREADS];
  __shared__ double wz[2 * MAX_D];
  const BEnt &b = tab[blockIdx.y];
  const int g = blockIdx.x;
  const int G = (int)(b.M < AP_GROUPS ? b.M : AP_GROUPS);
  if (g >= G) return;
  const int D = b.D, DD = D * D, tid = threadIdx.x;
  int P2 = 1;
  while (D * P2 * 2 <= OB_THREADS && D * P2 < b.M) P2 *= 2;
  const int Tp = D * P2;
  const double delta = OB_CLUSTER_REL * fmax(1.0, fmax(fabs(b.w[0]), fabs(b.w[b.M - 1])));
  int32_t nflag = 0;
  double acc[16];
  for (int k = 0; k < 16; ++k) acc[k] = 0.0;
  for (int64_t a = g; a < b.M; a += G) {
    const cd *col = b.HF + a * b.ld;
    double s = 0.0;
    if (tid < Tp)
      for (int64_t r = tid; r < b.M; r += Tp) s += cabs2(col[r]);
    red[tid] = s;
    __syncthreads();
    for (int h = P2 / 2; h >= 1; h >>= 1) {
      if (tid < D * h) red[tid] += red[tid + D * h];
      __syncthreads();
    }
    if (tid < D) {
      wz[tid] = red[tid];
      wz[MAX_D + tid] = cabs2(col[tid + (int64_t)D * b.s0]);
    }
    __syncthreads();
    for (int k = 0; k < 16; ++k) {
      const int e = tid + OB_THREADS * k;
      if (e >= DD) break;
      acc[k] += wz[e % D] * wz[MAX_D + e / D];
    }
    if (tid < 64) {                     // degenerate pairs (a, c > a) sharing weight on the zero site
      const double za = wave_sum(tid < D ? wz[MAX_D + tid] : 0.0);
      const double wa = b.w[a];
      for (int64_t c = a + 1; c < b.M && b.w[c] - wa <= delta; ++c) {
        const double zc = wave_sum(tid < D ? cabs2(b.HF[c * b.ld + tid + (int64_t)D * b.s0]) : 0.0);
        nflag += (za * zc > OB_SHARED_WEIGHT) ? 1 : 0;
      }
    }
    __syncthreads();
  }
  for (int k = 0; k < 16; ++k) {
    const int e = tid + OB_THREADS * k;
    if (e >= DD) break;
    b.part[(int64_t)g * DD + e] = acc[k];
  }
  if (tid == 0) b.flags[g] = nflag;
}

// P and status of problem blockIdx.x from its partials (fixed order).
__global__ void __launch_bounds__(OB_THREADS) ob_avgprob_sum(const BEnt *__restrict__ tab) {
  const BEnt &b = tab[blockIdx.x];
  const int G = (int)(b.M < AP_GROUPS ? b.M : AP_GROUPS);
  const int DD = b.D * b.D;
  for (int e = threadIdx.x; e < DD; e += OB_THREADS) {
    double s = 0.0;
    for (int g = 0; g < G; ++g) s += b.part[(int64_t)g * DD + e];
    b.P[e] = s;
  }
  if (threadIdx.x == 0) {
    int32_t f = 0;
    for (int g = 0; g < G; ++g) f |= (b.flags[g] != 0);
    *b.status = f ? MMF_ERR_DEGENERATE : 0;
  }
}

// ---------------------------------------------------------------- host side
struct BatchWs {
  BEnt *tab;
  std::vector<char *> prob;   // per-problem workspace bases
  size_t bytes;
};

inline size_t ob_prob_bytes(const FloqParams &fp, int32_t T) {
  Carver cv(nullptr);
  cv.take<cd>((size_t)fp.S * (T > 0 ? T : 1));
  cv.take<cd>((size_t)(T > 0 ? T : 1) * fp.M * fp.D);
  const int64_t G = fp.M < AP_GROUPS ? fp.M : AP_GROUPS;
  cv.take<double>((size_t)G * fp.D * fp.D);
  cv.take<int32_t>((size_t)G);
  return cv.used();
}

// Validates the problems (D <= 64, F <= BMAX_F, K <= BMAX_K) and fills fps.
static int batch_params(int64_t count, const mmf_problem *p, std::vector<FloqParams> &fps) {
  fps.resize((size_t)count);
  for (int64_t c = 0; c < count; ++c) {
    const int rc = problem_params_small_d(&p[c], 2, &fps[c]);
    if (rc) return rc;
    if (fps[c].F > BMAX_F || fps[c].K > BMAX_K) return MMF_ERR_TOO_LARGE;
  }
  return MMF_OK;
}

static BPack make_pack(const FloqParams &fp) {
  BPack e = {};
  e.D = fp.D; e.F = fp.F;
  for (int l = 0; l < BMAX_F; ++l) { e.N[l] = fp.N[l]; e.omega[l] = fp.omega[l]; }
  return e;
}

// The problem part of a table entry.
__device__ inline void unpack(const BPack &q, BEnt &e) {
  e.D = q.D; e.F = q.F;
  e.S = 1; e.s0 = 0;
  for (int l = 0; l < BMAX_F; ++l) {
    const bool in = l < q.F;
    e.N[l] = in ? q.N[l] : 0;
    e.omega[l] = in ? q.omega[l] : 0.0;
    e.radix[l] = 2 * e.N[l] + 1;
    e.s0 += e.N[l] * e.S;
    e.S *= e.radix[l];
  }
  e.M = q.D * e.S;
}

// Entries for the assembly.
struct BuildPack {
  BPack q;
  const cd *EV;
  cd *HF;
  int64_t ld;
  int32_t harm[BMAX_K];
  int8_t axis[BMAX_K];
  int32_t K;
};
__global__ void ob_set_build(BEnt *dst, TableChunk<BuildPack, 3840 / sizeof(BuildPack)> c) {
  const int i = threadIdx.x;
  if (i >= c.count) return;
  const BuildPack &v = c.v[i];
  BEnt e = {};
  unpack(v.q, e);
  e.K = v.K;
  for (int k = 0; k < BMAX_K; ++k) { e.axis[k] = v.axis[k]; e.harm[k] = v.harm[k]; }
  e.EV = v.EV; e.HF = v.HF; e.ld = v.ld;
  dst[i] = e;
}

// Entries for the observables; `base` is the problem's part of the workspace,
// carved as in ob_prob_bytes.
struct ObsPack {
  BPack q;
  cd *HF;
  int64_t ld;
  const double *w, *t;
  cd *U;
  double *P;
  char *base;
};
__global__ void ob_set_obs(BEnt *dst, int32_t *status, int32_t T, double t0,
                           TableChunk<ObsPack, 3840 / sizeof(ObsPack)> c) {
  const int i = threadIdx.x;
  if (i >= c.count) return;
  const ObsPack &v = c.v[i];
  BEnt e = {};
  unpack(v.q, e);
  e.T = T; e.t0 = t0;
  e.HF = v.HF; e.ld = v.ld; e.w = v.w; e.t = v.t; e.U = v.U; e.P = v.P;
  e.status = status + i;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    off = (off + 255) & ~(size_t)255;
    char *r = v.base + off;
    off += bytes;
    return r;
  };
  const int64_t G = e.M < AP_GROUPS ? e.M : AP_GROUPS;
  e.B = reinterpret_cast<cd *>(take((size_t)e.S * T * sizeof(cd)));
  e.Y = reinterpret_cast<cd *>(take((size_t)T * e.M * e.D * sizeof(cd)));
  e.part = reinterpret_cast<double *>(take((size_t)G * e.D * e.D * sizeof(double)));
  e.flags = reinterpret_cast<int32_t *>(take((size_t)G * sizeof(int32_t)));
  dst[i] = e;
}

}  // namespace mmf

using namespace mmf;

extern "C" int mmf_batched_workspace(int64_t count, const mmf_problem *p, int32_t T, size_t *bytes) {
  if (count < 0) return -1;
  if (count > 0 && !p) return -2;
  if (T < 0) return -3;
  if (!bytes) return -4;
  std::vector<FloqParams> fps;
  const int rc = batch_params(count, p, fps);
  if (rc) return rc;
  size_t b = ((size_t)(count > 0 ? count : 1) * sizeof(BEnt) + 255) & ~(size_t)255;
  for (int64_t c = 0; c < count; ++c) b += ob_prob_bytes(fps[c], T);
  *bytes = b;
  return MMF_OK;
}

extern "C" int mmf_build_floquet_batched(int64_t count, const mmf_problem *p, const mmf_z *const *EV,
                                         mmf_z *const *HF, const int64_t *ldh, void *work, size_t work_bytes,
                                         void *stream) {
  if (count < 0) return -1;
  if (count == 0) return MMF_OK;
  if (!p) return -2;
  std::vector<FloqParams> fps;
  int rc = batch_params(count, p, fps);
  if (rc) return rc;
  for (int64_t c = 0; c < count; ++c)
    if (!problem_hermitian(&p[c])) return -2;
  if (!EV) return -3;
  if (!HF) return -4;
  if (!ldh) return -5;
  for (int64_t c = 0; c < count; ++c) {
    if (!EV[c]) return -3;
    if (!HF[c]) return -4;
    if (ldh[c] < fps[c].M) return -5;
  }
  if (!work) return -6;
  if (work_bytes < (size_t)count * sizeof(BEnt)) return -7;
  hipStream_t st = (hipStream_t)stream;
  BEnt *tab = reinterpret_cast<BEnt *>(work);
  int64_t Mmax = 0;
  TableChunk<BuildPack, 3840 / sizeof(BuildPack)> ch;
  constexpr int64_t CH = 3840 / sizeof(BuildPack);
  for (int64_t c0 = 0; c0 < count; c0 += CH) {
    ch.count = (int32_t)(count - c0 < CH ? count - c0 : CH);
    for (int32_t i = 0; i < ch.count; ++i) {
      const FloqParams &fp = fps[c0 + i];
      BuildPack &v = ch.v[i];
      v.q = make_pack(fp);
      v.EV = reinterpret_cast<const cd *>(EV[c0 + i]);
      v.HF = reinterpret_cast<cd *>(HF[c0 + i]);
      v.ld = ldh[c0 + i];
      v.K = fp.K;
      for (int k = 0; k < BMAX_K; ++k) { v.axis[k] = (int8_t)fp.axis[k]; v.harm[k] = fp.harm[k]; }
      Mmax = fp.M > Mmax ? fp.M : Mmax;
    }
    hipLaunchKernelGGL(ob_set_build, dim3(1), dim3(64), 0, st, tab + c0, ch);
    MMF_LAUNCH_CHECK();
  }
  return assemble_batched_launch(tab, count, Mmax, st);
}

extern "C" int mmf_observables_batched(int64_t count, const mmf_problem *p, const mmf_z *const *Phi,
                                       const int64_t *ld, const double *const *w, double t0, int32_t T,
                                       const double *const *t, mmf_z *const *U, double *const *P,
                                       int32_t *dev_status, void *work, size_t work_bytes, void *stream) {
  if (count < 0) return -1;
  if (count == 0) return MMF_OK;
  if (!p) return -2;
  std::vector<FloqParams> fps;
  int rc = batch_params(count, p, fps);
  if (rc) return rc;
  if (!Phi) return -3;
  if (!ld) return -4;
  if (!w) return -5;
  if (T < 1) return -7;
  if (!t) return -8;
  if (!U) return -9;
  if (!P) return -10;
  for (int64_t c = 0; c < count; ++c) {
    if (!Phi[c]) return -3;
    if (ld[c] < fps[c].M) return -4;
    if (!w[c]) return -5;
    if (!t[c]) return -8;
    if (!U[c]) return -9;
    if (!P[c]) return -10;
    if ((int64_t)fps[c].D * T > 8 * OB_THREADS) return MMF_ERR_TOO_LARGE;    // D T outputs per projection workgroup
  }
  if (!dev_status) return -11;
  if (!work) return -12;
  size_t need = 0;
  mmf_batched_workspace(count, p, T, &need);
  if (work_bytes < need) return -13;
  char *cur = (char *)work + (((size_t)count * sizeof(BEnt) + 255) & ~(size_t)255);
  int64_t Smax_T = 0, Mmax = 0, proj = 0, qb = 1;   // largest grids of the batch
  int32_t Dmax = 0;
  hipStream_t st = (hipStream_t)stream;
  BEnt *tab = reinterpret_cast<BEnt *>(work);
  TableChunk<ObsPack, 3840 / sizeof(ObsPack)> ch;
  constexpr int64_t CH = 3840 / sizeof(ObsPack);
  for (int64_t c0 = 0; c0 < count; c0 += CH) {
    ch.count = (int32_t)(count - c0 < CH ? count - c0 : CH);
    for (int32_t i = 0; i < ch.count; ++i) {
      const int64_t c = c0 + i;
      const FloqParams &fp = fps[c];
      ObsPack &v = ch.v[i];
      v.q = make_pack(fp);
      v.HF = const_cast<cd *>(reinterpret_cast<const cd *>(Phi[c]));
      v.ld = ld[c];
      v.w = w[c];
      v.t = t[c];
      v.U = reinterpret_cast<cd *>(U[c]);
      v.P = P[c];
      v.base = cur;
      cur += ob_prob_bytes(fp, T);
      Smax_T = fp.S * T > Smax_T ? fp.S * T : Smax_T;
      Mmax = fp.M > Mmax ? fp.M : Mmax;
      Dmax = fp.D > Dmax ? fp.D : Dmax;
      proj = std::max(proj, (int64_t)cdiv(fp.M, ob_project_cols(fp.D, T)));
      qb = std::max(qb, (int64_t)cdiv(T, ob_contract_times(fp.D)));
    }
    hipLaunchKernelGGL(ob_set_obs, dim3(1), dim3(64), 0, st, tab + c0, dev_status + c0, T, t0, ch);
    MMF_LAUNCH_CHECK();
  }
  for (int64_t y0 = 0; y0 < count; y0 += 65535) {
    const unsigned yc = (unsigned)(count - y0 < 65535 ? count - y0 : 65535);
    hipLaunchKernelGGL(ob_phases, dim3(cdiv(Smax_T, OB_THREADS), yc), dim3(OB_THREADS), 0, st, tab + y0);
    MMF_LAUNCH_CHECK();
    const dim3 pg((unsigned)std::min<int64_t>(proj, OB_PROJ_GRID), yc), cg((unsigned)qb, yc);
    if ((int64_t)Dmax * T <= OB_THREADS)
      hipLaunchKernelGGL(ob_project<1>, pg, dim3(OB_THREADS), 0, st, tab + y0);
    else
      hipLaunchKernelGGL(ob_project<8>, pg, dim3(OB_THREADS), 0, st, tab + y0);
    MMF_LAUNCH_CHECK();
    if (Dmax <= 16)
      hipLaunchKernelGGL(ob_contract<1>, cg, dim3(OB_THREADS), 0, st, tab + y0);
    else
      hipLaunchKernelGGL(ob_contract<16>, cg, dim3(OB_THREADS), 0, st, tab + y0);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(ob_avgprob, dim3((unsigned)std::min<int64_t>(Mmax, AP_GROUPS), yc), dim3(OB_THREADS), 0, st, tab + y0);
    MMF_LAUNCH_CHECK();
    hipLaunchKernelGGL(ob_avgprob_sum, dim3(yc), dim3(OB_THREADS), 0, st, tab + y0);
    MMF_LAUNCH_CHECK();
  }
  return MMF_OK;
}
