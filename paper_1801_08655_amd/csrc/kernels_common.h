// Device helpers shared by the HIP kernels: complex arithmetic and loads.
#pragma once

#include <hip/hip_runtime.h>

#include "helm_internal.h"

namespace helm {
namespace kern {

template <typename T> using C_t = typename Cplx<T>::type;

template <typename C> __device__ __forceinline__ C cmake(double re, double im) {
  C z;
  z.x = re;
  z.y = im;
  return z;
}
template <typename C> __device__ __forceinline__ C czero() { return cmake<C>(0, 0); }

// Global-memory loads and stores through address-space-1 pointers.  A
// pointer read from a device structure is generic to the compiler, which
// then emits FLAT instructions; those also count against the LDS wait
// counter, so the LDS waits of an MFMA loop would wait for every global
// prefetch in flight.  Through these helpers the compiler emits
// global_load / global_store.  Only for pointers into device memory.
#define HELM_AS1 __attribute__((address_space(1)))
template <typename C> __device__ __forceinline__ C ld(const C* p) {
  typedef typename C::value_type E;
  typedef E V __attribute__((ext_vector_type(2)));
  const V v = *(const HELM_AS1 V*)p;
  C r;
  r.x = v.x;
  r.y = v.y;
  return r;
}
__device__ __forceinline__ int ld(const int* p) { return *(const HELM_AS1 int*)p; }

// A complex zero in device memory (room for complex128), the load address
// of the masked-off lanes of ld_or_zero.
static __device__ __align__(16) double kZeroC[2] = {0.0, 0.0};

// *p when ok, else zero, as one unconditional load (no branch), so that a
// run of such loads is issued back to back and waited for once.
template <typename C> __device__ __forceinline__ C ld_or_zero(bool ok, const C* p) {
  return ld(ok ? p : reinterpret_cast<const C*>(kZeroC));
}
template <typename C> __device__ __forceinline__ void st(C* p, C v) {
  typedef typename C::value_type E;
  typedef E V __attribute__((ext_vector_type(2)));
  V w;
  w.x = v.x;
  w.y = v.y;
  *(HELM_AS1 V*)p = w;
}
template <typename C> __device__ __forceinline__ C cadd(C a, C b) {
  C z; z.x = a.x + b.x; z.y = a.y + b.y; return z;
}
template <typename C> __device__ __forceinline__ C csub(C a, C b) {
  C z; z.x = a.x - b.x; z.y = a.y - b.y; return z;
}
template <typename C> __device__ __forceinline__ C cmul(C a, C b) {
  C z;
  z.x = a.x * b.x - a.y * b.y;
  z.y = a.x * b.y + a.y * b.x;
  return z;
}
template <typename C> __device__ __forceinline__ C cneg(C a) {
  C z; z.x = -a.x; z.y = -a.y; return z;
}
// a += b * c
template <typename C> __device__ __forceinline__ void cfma(C& a, C b, C c) {
  a.x += b.x * c.x - b.y * c.y;
  a.y += b.x * c.y + b.y * c.x;
}
// a -= b * c
template <typename C> __device__ __forceinline__ void cfms(C& a, C b, C c) {
  a.x -= b.x * c.x - b.y * c.y;
  a.y -= b.x * c.y + b.y * c.x;
}
// a / b with scaling against overflow (Smith's method)
template <typename C> __device__ __forceinline__ C cdiv(C a, C b) {
  C z;
  if (fabs((double)b.x) >= fabs((double)b.y)) {
    auto r = b.y / b.x;
    auto d = b.x + b.y * r;
    z.x = (a.x + a.y * r) / d;
    z.y = (a.y - a.x * r) / d;
  } else {
    auto r = b.x / b.y;
    auto d = b.x * r + b.y;
    z.x = (a.x * r + a.y) / d;
    z.y = (a.y * r - a.x) / d;
  }
  return z;
}
template <typename C> __device__ __forceinline__ double cabs2(C a) {
  return (double)a.x * a.x + (double)a.y * a.y;
}

__device__ __forceinline__ double2 to_d2(float2 a) { return make_double2(a.x, a.y); }
__device__ __forceinline__ double2 to_d2(double2 a) { return a; }
template <typename C> __device__ __forceinline__ C from_d2(double2 a);
template <> __device__ __forceinline__ float2 from_d2<float2>(double2 a) {
  return make_float2((float)a.x, (float)a.y);
}
template <> __device__ __forceinline__ double2 from_d2<double2>(double2 a) { return a; }

// v of one lane (the same lane for the whole wave)
template <typename T> __device__ __forceinline__ T lane_read(T v, int lane);
template <> __device__ __forceinline__ float lane_read<float>(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
template <> __device__ __forceinline__ double lane_read<double>(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Launches over variable-size items (fronts, their tiles and chunks) index
// their blocks through a tile map built on the host: entry t holds the item
// of block t and the block's index within that item, so a block finds its
// work with one load.

constexpr int GT = 64;   // tile edge (complex elements)
constexpr int FWD_BM = 64;   // row tile of the forward substitution GEMM
constexpr int RT = 16;       // row tile of the gather / split-K reduction kernels

}  // namespace kern
}  // namespace helm
