// Quaternion, tangent and sphere-against-box derivatives of the adjoint kernels.  Included after the vector helpers
// (V3, mk, add, ...) of the including source.
#pragma once

namespace ags {
namespace {

// Hamilton product, xyzw
template <typename R>
__device__ __forceinline__ void qmul(const R* a, const R* b, R* o) {
  o[0] = a[3] * b[0] + a[0] * b[3] + a[1] * b[2] - a[2] * b[1];
  o[1] = a[3] * b[1] - a[0] * b[2] + a[1] * b[3] + a[2] * b[0];
  o[2] = a[3] * b[2] + a[0] * b[1] - a[1] * b[0] + a[2] * b[3];
  o[3] = a[3] * b[3] - a[0] * b[0] - a[1] * b[1] - a[2] * b[2];
}
// rotation increment Exp(theta) = (sin(|t|/2) t/|t|, cos(|t|/2)); (t/2, 1) below 1e-8
template <typename R>
__device__ __forceinline__ void dq_of(V3<R> th, R* dq) {
  const R ang = sqrt_(dot(th, th));
  if (ang < R(1e-8)) {
    dq[0] = R(0.5) * th.x; dq[1] = R(0.5) * th.y; dq[2] = R(0.5) * th.z; dq[3] = R(1);
  } else {
    R s, c;
    sincos_(R(0.5) * ang, &s, &c);
    const R sc = s / ang;
    dq[0] = th.x * sc; dq[1] = th.y * sc; dq[2] = th.z * sc; dq[3] = c;
  }
}
template <typename R>
__device__ __forceinline__ V3<R> dq_adj(V3<R> th, const R* dqb) {
  const R ang = sqrt_(dot(th, th));
  const V3<R> gv = mk(dqb[0], dqb[1], dqb[2]);
  if (ang < R(1e-8)) return mul(gv, R(0.5));
  R s, c;
  sincos_(R(0.5) * ang, &s, &c);
  const R sc = s / ang;
  const R dsc = (R(0.5) * c * ang - s) / (ang * ang);  // d(sin(a/2)/a)/da
  return add(mul(gv, sc), mul(th, (dot(th, gv) * dsc - R(0.5) * s * dqb[3]) / ang));
}

// tangent basis of a contact normal: t1 = normalised projection of the world axis least aligned with n
// (lowest index on ties), t2 = n x t1 (the rule of the step kernel)
template <typename R>
__device__ __forceinline__ int tangents(V3<R> n, V3<R>& t1, V3<R>& t2, V3<R>& t) {
  const R ax = n.x < R(0) ? -n.x : n.x, ay = n.y < R(0) ? -n.y : n.y, az = n.z < R(0) ? -n.z : n.z;
  int k = 0;
  R best = ax;
  if (ay < best) {
    best = ay;
    k = 1;
  }
  if (az < best) k = 2;
  const V3<R> e = k == 0 ? mk(R(1), R(0), R(0)) : (k == 1 ? mk(R(0), R(1), R(0)) : mk(R(0), R(0), R(1)));
  t = sub(e, mul(n, dot(n, e)));
  t1 = mul(t, R(1) / sqrt_(dot(t, t)));
  t2 = cross(n, t1);
  return k;
}
// adjoint of n through (t1, t2) = tangents(n)
template <typename R>
__device__ __forceinline__ V3<R> tangents_adj(V3<R> n, V3<R> t1b, V3<R> t2b) {
  V3<R> t1, t2, t;
  const int k = tangents(n, t1, t2, t);
  V3<R> nb = cross(t1, t2b);
  t1b = add(t1b, cross(t2b, n));
  const V3<R> tb = mul(sub(t1b, mul(t1, dot(t1, t1b))), R(1) / sqrt_(dot(t, t)));
  const R nk = k == 0 ? n.x : (k == 1 ? n.y : n.z);
  nb = sub(nb, mul(tb, nk));
  const R ntb = dot(n, tb);
  if (k == 0) nb.x -= ntb;
  else if (k == 1) nb.y -= ntb;
  else nb.z -= ntb;
  return nb;
}
// sphere (centre c, radius r) against a box (rotation Rb row-major, centre b, half extents hb): signed
// distance and normal (from the box towards the sphere) by the closest point, or the face of least
// penetration when the centre is inside (the step kernel's rule).  G (optional) = dn / d(c - moving box
// point), row-major: Rb (1 - nl nl^T) diag(clamped axes) Rb^T / |d| outside, 0 inside.
template <typename R>
__device__ __forceinline__ void sphere_box(V3<R> c, const R* Rb, V3<R> b, V3<R> hb, R rad, R& phi, V3<R>& n, R* G) {
  const V3<R> u = sub(c, b);
  const V3<R> xl = mk(Rb[0] * u.x + Rb[3] * u.y + Rb[6] * u.z, Rb[1] * u.x + Rb[4] * u.y + Rb[7] * u.z,
                      Rb[2] * u.x + Rb[5] * u.y + Rb[8] * u.z);
  const V3<R> ql = mk(fmin(fmax(xl.x, -hb.x), hb.x), fmin(fmax(xl.y, -hb.y), hb.y), fmin(fmax(xl.z, -hb.z), hb.z));
  const bool inside = ql.x == xl.x && ql.y == xl.y && ql.z == xl.z;
  const V3<R> dl = sub(xl, ql);
  const R dn = sqrt_(dot(dl, dl));
  V3<R> nl;
  if (!inside && dn > R(1e-12)) {
    phi = dn - rad;
    nl = mul(dl, R(1) / dn);
    if (G) {
      const R m[3] = {xl.x != ql.x ? R(1) : R(0), xl.y != ql.y ? R(1) : R(0), xl.z != ql.z ? R(1) : R(0)};
      const R nv[3] = {nl.x, nl.y, nl.z};
      R Lc[9];  // (1 - nl nl^T) diag(m) / dn in box coordinates
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) Lc[3 * i + j] = ((i == j ? R(1) : R(0)) - nv[i] * nv[j]) * m[j] / dn;
      R T[9];  // Rb Lc
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) T[3 * i + j] = Rb[3 * i] * Lc[j] + Rb[3 * i + 1] * Lc[3 + j] + Rb[3 * i + 2] * Lc[6 + j];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) G[3 * i + j] = T[3 * i] * Rb[3 * j] + T[3 * i + 1] * Rb[3 * j + 1] + T[3 * i + 2] * Rb[3 * j + 2];
    }
  } else {
    const R p0 = hb.x - (xl.x < R(0) ? -xl.x : xl.x), p1 = hb.y - (xl.y < R(0) ? -xl.y : xl.y),
            p2 = hb.z - (xl.z < R(0) ? -xl.z : xl.z);
    int kb = 0;
    R pb = p0, xb = xl.x;
    if (p1 < pb) { kb = 1; pb = p1; xb = xl.y; }
    if (p2 < pb) { kb = 2; pb = p2; xb = xl.z; }
    const R sg = xb >= R(0) ? R(1) : R(-1);
    nl = kb == 0 ? mk(sg, R(0), R(0)) : (kb == 1 ? mk(R(0), sg, R(0)) : mk(R(0), R(0), sg));
    phi = -pb - rad;
    if (G) {
#pragma unroll
      for (int k = 0; k < 9; ++k) G[k] = R(0);
    }
  }
  n = mv(Rb, nl);
}

}  // namespace
}  // namespace ags
