// Device helpers shared by the kernel files: typed views of device vectors, the FP32 phase,
// the `active` flag of a CG.
#pragma once

#include "hub_internal.h"

namespace hub {
namespace {

template <typename R> struct V2;
template <> struct V2<double> { using T = double2; };
template <> struct V2<float> { using T = float2; };

template <typename C> __device__ __forceinline__ C cz() { C z; z.x = 0; z.y = 0; return z; }

template <typename R, typename C>
__device__ __forceinline__ R norm2(C a) { return a.x * a.x + a.y * a.y; }

// Views of device vectors in the global address space.  Pointers read from a
// descriptor are generic; accessing them through these views makes the compiler
// emit global_* instead of flat_* memory instructions.
#define HUB_GAS __attribute__((address_space(1)))
typedef double hub_d2v __attribute__((ext_vector_type(2)));
typedef float hub_f2v __attribute__((ext_vector_type(2)));
template <typename C> struct Vec;
template <> struct Vec<double2> {
  HUB_GAS hub_d2v* p;
  __device__ __forceinline__ explicit Vec(const void* q) : p((HUB_GAS hub_d2v*)q) {}
  __device__ __forceinline__ double2 operator[](int k) const {
    const hub_d2v v = p[k];
    double2 r;
    r.x = v.x;
    r.y = v.y;
    return r;
  }
  __device__ __forceinline__ void set(int k, double2 a) const {
    hub_d2v v;
    v.x = a.x;
    v.y = a.y;
    p[k] = v;
  }
};
typedef float hub_f4v __attribute__((ext_vector_type(4)));
// Two consecutive complex64 values (sites k, k+1 with k even: one 16-byte access).
struct C64x2 {
  float2 a, b;
};
template <> struct Vec<float2> {
  HUB_GAS hub_f2v* p;
  __device__ __forceinline__ explicit Vec(const void* q) : p((HUB_GAS hub_f2v*)q) {}
  __device__ __forceinline__ C64x2 pair(int k) const {
    const hub_f4v v = ((HUB_GAS hub_f4v*)p)[k >> 1];
    C64x2 r;
    r.a.x = v.x;
    r.a.y = v.y;
    r.b.x = v.z;
    r.b.y = v.w;
    return r;
  }
  __device__ __forceinline__ void set_pair(int k, C64x2 a) const {
    hub_f4v v;
    v.x = a.a.x;
    v.y = a.a.y;
    v.z = a.b.x;
    v.w = a.b.y;
    ((HUB_GAS hub_f4v*)p)[k >> 1] = v;
  }
  __device__ __forceinline__ float2 operator[](int k) const {
    const hub_f2v v = p[k];
    float2 r;
    r.x = v.x;
    r.y = v.y;
    return r;
  }
  __device__ __forceinline__ void set(int k, float2 a) const {
    hub_f2v v;
    v.x = a.x;
    v.y = a.y;
    p[k] = v;
  }
};
template <typename T> struct Real {
  HUB_GAS T* p;
  __device__ __forceinline__ explicit Real(const void* q) : p((HUB_GAS T*)q) {}
  __device__ __forceinline__ T operator[](int k) const { return p[k]; }
  __device__ __forceinline__ void set(int k, T v) const { p[k] = v; }
  // values at k, k+1 (k even): one 8-byte access for float
  __device__ __forceinline__ hub_f2v pair(int k) const { return ((HUB_GAS hub_f2v*)p)[k >> 1]; }
};

// cos x and sin x in FP32 for the complex64 solver kernels, |x| <= pi in practice (the
// angle is reduced when the solve starts): r = x - q pi/2 with q the integer nearest
// 2x/pi (difference and product in FP64, exact far below FP32 rounding), cos r and
// sin r on |r| <= pi/4 from their Taylor series through degree 10 and 9 (the first
// omitted terms are below 2.5e-9, under half an FP32 ulp), then (cos r, sin r) turned
// by q quarter turns.  Error against e^{ix}: about one FP32 ulp.
__device__ __forceinline__ void cis32(float x, float& c, float& s) {
  const float q = rintf(x * 0.636619772f);
  const float r = (float)fma(-(double)q, 1.5707963267948966, (double)x);
  const float r2 = r * r;
  float ps = fmaf(r2, 2.75573192e-6f, -1.98412698e-4f);  // 1/9!, -1/7!
  ps = fmaf(ps, r2, 8.33333333e-3f);                      // 1/5!
  ps = fmaf(ps, r2, -1.66666667e-1f);                     // -1/3!
  const float sr = fmaf(ps * r2, r, r);
  float pc = fmaf(r2, -2.75573192e-7f, 2.48015873e-5f);  // -1/10!, 1/8!
  pc = fmaf(pc, r2, -1.38888889e-3f);                     // -1/6!
  pc = fmaf(pc, r2, 4.16666667e-2f);                      // 1/4!
  pc = fmaf(pc, r2, -0.5f);
  const float cr = fmaf(pc, r2, 1.0f);
  const int k = (int)q & 3;
  c = (k == 0) ? cr : (k == 1) ? -sr : (k == 2) ? -cr : sr;
  s = (k == 0) ? sr : (k == 1) ? cr : (k == 2) ? -sr : -cr;
}
__device__ __forceinline__ int load_active(Scal* sc) {
  return __hip_atomic_load(&sc->active, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_active(Scal* sc, int v) {
  __hip_atomic_store(&sc->active, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sums within a wave by data-parallel primitives (row shifts, then row broadcasts): a few
// cycles per step where a shuffle through LDS takes some sixty.  dpp_row leaves the sum of
// lanes 0..15 in lane 15 (of each row of 16), dpp_wave the sum of all in lane 63.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xf, false);
  return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename T>
__device__ __forceinline__ T dpp_row(T v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  return dpp_add<0x118, 0xf>(v);
}
template <typename T>
__device__ __forceinline__ T dpp_wave(T v) {
  v = dpp_row(v);
  v = dpp_add<0x142, 0xa>(v);
  return dpp_add<0x143, 0xc>(v);
}

// Words exchanged between workgroups inside a kernel: written through to and read past the
// L2 caches of the XCDs.  drain() waits until this wave's stores have arrived there (or, for
// system-scope stores, in host memory); a counter increment after it publishes them.
__device__ __forceinline__ void put_agent(double* p, double v) {
  __hip_atomic_store((unsigned long long*)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_agent(const double* p) {
  return __longlong_as_double((long long)__hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

}  // namespace
}  // namespace hub
