// Shared device/host helpers of libmmf (internal header, not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "mmf.h"

#define MMF_HIP_TRY(expr)                                   \
  do {                                                      \
    hipError_t _e = (expr);                                 \
    if (_e != hipSuccess) return MMF_ERR_HIP;               \
  } while (0)

namespace mmf {
// After every kernel launch: nonzero if the launch failed.  With the opt-in
// profiling throttle (mmf_profile_sync_every) it also waits for the device
// every n launches.
int launch_check();
}  // namespace mmf

#define MMF_LAUNCH_CHECK()                                  \
  do {                                                      \
    if (mmf::launch_check() != 0) return MMF_ERR_HIP;       \
  } while (0)
// the same with a clean-up statement before the error return
#define MMF_LAUNCH_CHECK_OR(cleanup)                        \
  do {                                                      \
    if (mmf::launch_check() != 0) {                         \
      cleanup;                                              \
      return MMF_ERR_HIP;                                   \
    }                                                       \
  } while (0)

// Global-memory pointer.  A pointer read from a device table is generic to the
// compiler, and a generic (FLAT) access counts against the same wait counter as
// LDS and scalar loads, so every wait for an LDS read would also wait for the
// HBM loads and stores still in flight.  Kernels view such pointers through
// this qualifier (all device buffers of the library are global memory).  The
// host pass, which also reads device code, takes it as a plain pointer.
#if defined(__HIP_DEVICE_COMPILE__)
#define MMF_GLOBAL __attribute__((address_space(1)))
#else
#define MMF_GLOBAL
#endif

namespace mmf {

// Value behind a global pointer (the operands of a conditional expression
// cannot mix address spaces).
template <typename T>
__device__ __forceinline__ T gload(const MMF_GLOBAL T *p) { return *p; }

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));

// Complex arithmetic on interleaved (re, im) pairs of R = double or float.
template <typename R>
struct alignas(2 * sizeof(R)) cx {
  R re, im;
};
typedef cx<double> cd;
typedef cx<float> cf;

template <typename R>
__host__ __device__ inline cx<R> cmk(R r, R i) { cx<R> z; z.re = r; z.im = i; return z; }
__host__ __device__ inline cd cmake(double r, double i) { return cmk<double>(r, i); }
template <typename R>
__device__ inline cx<R> cadd(cx<R> a, cx<R> b) { return cmk<R>(a.re + b.re, a.im + b.im); }
template <typename R>
__device__ inline cx<R> csub(cx<R> a, cx<R> b) { return cmk<R>(a.re - b.re, a.im - b.im); }
template <typename R>
__device__ inline cx<R> cmul(cx<R> a, cx<R> b) {
  return cmk<R>(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
// conj(a) * b
template <typename R>
__device__ inline cx<R> cmulc(cx<R> a, cx<R> b) {
  return cmk<R>(a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re);
}
// x - a b in four fused operations (not left to contraction: the same bits wherever it is used)
__device__ inline cd cfnma(cd x, cd a, cd b) {
  return cmake(fma(a.im, b.im, fma(-a.re, b.re, x.re)), fma(-a.im, b.re, fma(-a.re, b.im, x.im)));
}
template <typename R>
__device__ inline cx<R> cconj(cx<R> a) { return cmk<R>(a.re, -a.im); }
template <typename R>
__device__ inline cx<R> cscale(cx<R> a, R s) { return cmk<R>(a.re * s, a.im * s); }
template <typename R>
__device__ inline R cabs2(cx<R> a) { return a.re * a.re + a.im * a.im; }

__device__ inline cd ldz(const mmf_z *p) {
  const double2 v = *reinterpret_cast<const double2 *>(p);
  return cmake(v.x, v.y);
}
__device__ inline void stz(mmf_z *p, cd v) {
  double2 t; t.x = v.re; t.y = v.im;
  *reinterpret_cast<double2 *>(p) = t;
}
// generic complex load/store on cx<R> storage (16 B for double, 8 B for float)
template <typename R>
__device__ inline cx<R> ldc(const cx<R> *p) { return *p; }
template <typename R>
__device__ inline void stc(cx<R> *p, cx<R> v) { *p = v; }

// Lane exchanges on the vector unit (DPP row operations, permlane swaps)
// instead of ds_bpermute: a 64-lane sum takes 6 steps of a few cycles each,
// where every __shfl_xor step is a round trip through the LDS crossbar.
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
  return __hiloint2double(dpp_mov<CTRL>(__double2hiint(v)), dpp_mov<CTRL>(__double2loint(v)));
}
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) { return __int_as_float(dpp_mov<CTRL>(__float_as_int(v))); }

// Sum over each row of 16 lanes, in every lane of the row.
template <typename R>
__device__ __forceinline__ R row16_sum(R v) {
  v += dpp_mov<0xB1>(v);     // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);     // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);    // row_half_mirror
  v += dpp_mov<0x140>(v);    // row_mirror
  return v;
}

// Sum over the four rows of lanes (lanes l, l ^ 16, l ^ 32, l ^ 48), in every lane.
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ void swap16(int v, int &a, int &b) {
  const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  a = (int)r[0]; b = (int)r[1];
}
__device__ __forceinline__ void swap32(int v, int &a, int &b) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  a = (int)r[0]; b = (int)r[1];
}
#else
__device__ inline void swap16(int v, int &a, int &b) { a = b = v; }
__device__ inline void swap32(int v, int &a, int &b) { a = b = v; }
#endif
__device__ __forceinline__ double rows_sum(double v) {
  int h0, h1, l0, l1;
  swap16(__double2hiint(v), h0, h1);
  swap16(__double2loint(v), l0, l1);
  v = __hiloint2double(h0, l0) + __hiloint2double(h1, l1);
  swap32(__double2hiint(v), h0, h1);
  swap32(__double2loint(v), l0, l1);
  return __hiloint2double(h0, l0) + __hiloint2double(h1, l1);
}
__device__ __forceinline__ float rows_sum(float v) {
  int a, b;
  swap16(__float_as_int(v), a, b);
  v = __int_as_float(a) + __int_as_float(b);
  swap32(__float_as_int(v), a, b);
  return __int_as_float(a) + __int_as_float(b);
}

// Value of lane u, in every lane (u uniform).
__device__ __forceinline__ double lane_get(double v, int u) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), u),
                          __builtin_amdgcn_readlane(__double2loint(v), u));
}
__device__ __forceinline__ float lane_get(float v, int u) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), u));
}
__device__ __forceinline__ cd lane_get(cd v, int u) { return cmake(lane_get(v.re, u), lane_get(v.im, u)); }

// Folds of two values: the lower (fold32: lanes < 32, fold16: even rows of 16)
// lanes receive a summed over both halves, the others b.
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ double lanes_fold32(double a, double b) {
  const auto l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double lanes_fold16(double a, double b) {
  const auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ float lanes_fold32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float lanes_fold16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
#else
template <typename R> __device__ inline R lanes_fold32(R a, R b) { return a + b; }
template <typename R> __device__ inline R lanes_fold16(R a, R b) { return a + b; }
#endif

// Wavefront-wide sum (all 64 lanes active), the same value in every lane.
__device__ __forceinline__ double wave_sum(double v) { return rows_sum(row16_sum(v)); }
__device__ __forceinline__ float wave_sum(float v) { return rows_sum(row16_sum(v)); }
__device__ inline double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

// 256-byte aligned carving of a caller workspace.
struct Carver {
  char *base;
  size_t off;
  explicit Carver(void *p) : base((char *)p), off(0) {}
  template <class T>
  T *take(size_t count) {
    off = (off + 255) & ~(size_t)255;
    T *r = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += count * sizeof(T);
    return r;
  }
  size_t used() const { return (off + 255) & ~(size_t)255; }
};

}  // namespace mmf
