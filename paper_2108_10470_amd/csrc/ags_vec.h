// Scalar, vector and lane helpers of the step kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace ags {
namespace {

// ---------------------------------------------------------------- scalar helpers
__device__ __forceinline__ float rsqrt_(float x) { return 1.0f / sqrtf(x); }
__device__ __forceinline__ double rsqrt_(double x) { return 1.0 / sqrt(x); }
__device__ __forceinline__ float sqrt_(float x) { return sqrtf(x); }
__device__ __forceinline__ double sqrt_(double x) { return sqrt(x); }
__device__ __forceinline__ float min_(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double min_(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float max_(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double max_(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float abs_(float a) { return fabsf(a); }
__device__ __forceinline__ double abs_(double a) { return fabs(a); }
__device__ __forceinline__ void sincos_(float x, float* s, float* c) { sincosf(x, s, c); }
__device__ __forceinline__ void sincos_(double x, double* s, double* c) { sincos(x, s, c); }

template <typename R>
struct V3 {
  R x, y, z;
};
template <typename R>
__device__ __forceinline__ V3<R> mk(R x, R y, R z) {
  return {x, y, z};
}
template <typename R>
__device__ __forceinline__ V3<R> add(V3<R> a, V3<R> b) {
  return {a.x + b.x, a.y + b.y, a.z + b.z};
}
template <typename R>
__device__ __forceinline__ V3<R> sub(V3<R> a, V3<R> b) {
  return {a.x - b.x, a.y - b.y, a.z - b.z};
}
template <typename R>
__device__ __forceinline__ V3<R> mul(V3<R> a, R s) {
  return {a.x * s, a.y * s, a.z * s};
}
template <typename R>
__device__ __forceinline__ R dot(V3<R> a, V3<R> b) {
  return a.x * b.x + a.y * b.y + a.z * b.z;
}
template <typename R>
__device__ __forceinline__ V3<R> cross(V3<R> a, V3<R> b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
template <typename R, typename P>
__device__ __forceinline__ V3<R> ld3(const P& p) {
  return {R(p[0]), R(p[1]), R(p[2])};
}
template <typename R, typename P>
__device__ __forceinline__ void st3(const P& p, V3<R> v) {
  p[0] = v.x;
  p[1] = v.y;
  p[2] = v.z;
}
template <typename R>
__device__ __forceinline__ void st3(R* p, V3<R> v) {
  p[0] = v.x;
  p[1] = v.y;
  p[2] = v.z;
}
// 3x3 row-major helpers
template <typename R, typename P>
__device__ __forceinline__ V3<R> mv(const P& M, V3<R> v) {
  return {M[0] * v.x + M[1] * v.y + M[2] * v.z, M[3] * v.x + M[4] * v.y + M[5] * v.z,
          M[6] * v.x + M[7] * v.y + M[8] * v.z};
}
template <typename R, typename P>
__device__ __forceinline__ V3<R> mtv(const P& M, V3<R> v) {
  return {M[0] * v.x + M[3] * v.y + M[6] * v.z, M[1] * v.x + M[4] * v.y + M[7] * v.z,
          M[2] * v.x + M[5] * v.y + M[8] * v.z};
}
template <typename PA, typename PB, typename R>
__device__ __forceinline__ void mm3(const PA& A, const PB& B, R* C) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) C[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
}

__device__ __forceinline__ unsigned long long lanes_below(int t) { return (1ull << t) - 1ull; }
// value of x in lane l (l uniform across the wave)
__device__ __forceinline__ int lane_read(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ float lane_read(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ double lane_read(double x, int l) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)(v & 0xffffffffll), l);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// tangent basis of a contact normal: t1 = normalised projection of the world axis least aligned with n
// (lowest index on ties), t2 = n x t1
template <typename R>
__device__ __forceinline__ void tangents(V3<R> n, V3<R>& t1, V3<R>& t2) {
  R ax = abs_(n.x), ay = abs_(n.y), az = abs_(n.z);
  int k = 0;
  R best = ax;
  if (ay < best) {
    best = ay;
    k = 1;
  }
  if (az < best) k = 2;
  V3<R> e = k == 0 ? mk(R(1), R(0), R(0)) : (k == 1 ? mk(R(0), R(1), R(0)) : mk(R(0), R(0), R(1)));
  V3<R> t = sub(e, mul(n, dot(n, e)));
  t1 = mul(t, rsqrt_(dot(t, t)));
  t2 = cross(n, t1);
}

// clamp to [lo, hi] (lo <= hi): one median-of-three in FP32
__device__ __forceinline__ float clamp_(float x, float lo, float hi) { return __builtin_amdgcn_fmed3f(x, lo, hi); }
// in FP64 a max then a min, written out: fmin/fmax of loop-carried bounds compile to two more instructions per
// call that quiet signalling NaNs, which no operand here can be
__device__ __forceinline__ double clamp_(double x, double lo, double hi) {
  double r;
  asm("v_max_f64 %0, %1, %2\n\tv_min_f64 %0, %0, %3" : "=&v"(r) : "v"(x), "v"(lo), "v"(hi));
  return r;
}

// upper impulse bound of rows without one (contact normals, limits): far above any impulse, finite so that
// the friction-bound arithmetic of the register Gauss-Seidel stays free of infinities
constexpr double kOpenBound = 1e30;

// bias of a limit or contact-normal row from its position error C: speculative C / h when separated, the
// Baumgarte fraction beta C / h when penetrating
template <typename R>
__device__ __forceinline__ R row_bias(R C, R h, R beta) {
  return C >= R(0) ? C / h : beta * C / h;
}

// rotation matrix (row-major) of a unit quaternion xyzw
template <typename R>
__device__ __forceinline__ void quat_R(R qx, R qy, R qz, R qw, R* M) {
  const R one = R(1), two = R(2);
  M[0] = one - two * (qy * qy + qz * qz); M[1] = two * (qx * qy - qz * qw); M[2] = two * (qx * qz + qy * qw);
  M[3] = two * (qx * qy + qz * qw); M[4] = one - two * (qx * qx + qz * qz); M[5] = two * (qy * qz - qx * qw);
  M[6] = two * (qx * qz - qy * qw); M[7] = two * (qy * qz + qx * qw); M[8] = one - two * (qx * qx + qy * qy);
}
template <typename R, typename P>
__device__ __forceinline__ void quat_R(const P& q, R* M) {
  quat_R(R(q[0]), R(q[1]), R(q[2]), R(q[3]), M);
}

}  // namespace
}  // namespace ags
