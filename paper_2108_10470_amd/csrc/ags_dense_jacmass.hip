// Dense form of the Jacobian and mass-matrix tensors (ags_jacmass.hip states them) for models of at most 31 generalized
// velocities and 32 links: one wavefront per environment, FP64 with FP32 outputs.
//
// It is bound by instruction issue, then by the 17 KB that an environment of the humanoid-like model writes.  The general
// form walks the tree level by level with barriers, sums subtrees link by link and divides for every output's place.
// Here poses come by pointer jumping, subtree sums and M = F S^T from the matrix cores (the dense step's pieces), and the
// outputs' inner dimension is a lane's column: its axis stays in registers while the links go by, two per round.
// 4096 humanoid-like environments (71 MB written): 22 us per call, 3.2 TB/s; the general form's two wavefronts per
// environment take 46 us.
#include "ags_dense_ops.h"

namespace ags {
namespace {

template <int NC>
struct JacLds {
  static constexpr int t_la = 0, t_lcm = NC, t_ccm = 2 * NC;  // ints
  static constexpr int qj = 3 * NC / 2, org = qj + NC, S = org + 4, pose = S + 6 * NC, Fm = pose + kDensePose * NC,
                       X = Fm + 6 * NC, x_words = kDenseXStride * NC > NC * (NC + 1) / 2 ? kDenseXStride * NC : NC * (NC + 1) / 2,
                       root = X + x_words;  // 13 words per actor
};

template <int NC>
__global__ __launch_bounds__(64) void dense_jacmass_kernel(JacMassArgs) {
  using L = JacLds<NC>;
  const auto P = (Cp<JacMassArgs>)__builtin_amdgcn_kernarg_segment_ptr();
  const Lp<R> sm = (Lp<R>)g_dense_lds;
  const Lp<int> si_ = (Lp<int>)g_dense_lds;
  const int lane = threadIdx.x, ei = blockIdx.x;
  const int env = __builtin_amdgcn_readfirstlane(gp(P->env_list)[ei]);
  const int nl = P->m.n_links, nv = P->m.n_v, na = P->m.n_actors;
  const int abase = gp(P->env_actor_base)[env], dbase = gp(P->env_dof_base)[env];
  const Lp<int> la = si_ + L::t_la, lcm = si_ + L::t_lcm, ccm = si_ + L::t_ccm;
  const Lp<R> qj = sm + L::qj, org = sm + L::org, S = sm + L::S, pose = sm + L::pose, Fm = sm + L::Fm, X = sm + L::X,
              root = sm + L::root;
  LinkLane lk{0, -1};
  ColLane cl{0};
  for (int k = lane; k < 13 * na; k += 64) root[k] = R(gp(P->root_state)[(long long)abase * 13 + k]);
  lane_tables<NC>(&P->m, lane, lk, cl, la, lcm, ccm);
  if (cl.joint()) qj[cl.dof()] = R(gp(P->dof_state)[2ll * (dbase + cl.dof())]);
  wsync();
  if (lane < 3) org[lane] = root[lane];
  wsync();
  R Q[4];
  V3<R> o;
  const auto lf = gp(P->m.lf) + (lk.is() ? lane : 0) * LF_COLS;
  poses<NC>(lf, lk, P->m.n_jump, root, qj, pose, S, org, nv, lane, Q, o);
  const int col = lane & 31, half = lane >> 5;
  if (P->mass) {
    R w[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) w[q] = R(0);
    if (lk.is()) {
      link_body(lf, Q, o).spatial(w);
      if (P->mass_scale) {
        const R f = R(gp(P->mass_scale)[gp(P->env_body_base)[env] + lane]);
#pragma unroll
        for (int q = 0; q < 10; ++q) w[q] *= f;
      }
    }
    // links with non-finite terms stay out of the products with 0/1 matrices (0 x NaN); the sums they belong to get NaN
    R off = R(0);
#pragma unroll
    for (int q = 0; q < 10; ++q) off += R(0) * w[q];
    const unsigned bad = (unsigned)__ballot(!(off == R(0)));
    if (lane < NC) {
#pragma unroll
      for (int q = 0; q < 16; ++q) X[kDenseXStride * lane + q] = (bad >> lane) & 1u ? R(0) : w[q];
    }
    wsync();
    subtree_sum<NC>(X, la, lane, X, la, 0);
    for (unsigned m = bad; m; m &= m - 1) {
      const int above = la[__ffs(m) - 1];
      if (lane < NC && ((above >> lane) & 1)) X[kDenseXStride * lane] = X[kDenseXStride * lane + 1] = R(NAN);
      wsync();
    }
    if (lane < NC) st6(Fm + 6 * lane, comp_mul(X + kDenseXStride * cl.link(), ld6(S + 6 * lane)));
    wsync();
    mass_matrix<NC>(Fm, S, ccm, X, lane);
    const auto out = gp(P->mass) + (long long)ei * nv * nv;
    if (col < nv)
      for (int k = half; k < nv; k += 2) {
        const int i = max(k, col), j = min(k, col);
        out[k * nv + col] = (float)X[i * (i + 1) / 2 + j];
      }
  }
  if (P->jac) {
    // column k moves link b: b's origin moves at v_k + w_k x o_b, b turns at w_k
    const auto out = gp(P->jac) + (long long)ei * nl * 6 * nv;
    const SV s = ld6(S + 6 * min(col, NC - 1));
    if (col < nv)
      for (int b = half; b < nl; b += 2) {
        const bool on = (lcm[b] >> col) & 1;
        const V3<R> v = add(s.v, cross(s.w, ld3<R>(pose + kDensePose * b + 4)));
        const auto p = out + b * 6 * nv + col;
        p[0] = on ? (float)v.x : 0.0f;
        p[nv] = on ? (float)v.y : 0.0f;
        p[2 * nv] = on ? (float)v.z : 0.0f;
        p[3 * nv] = on ? (float)s.w.x : 0.0f;
        p[4 * nv] = on ? (float)s.w.y : 0.0f;
        p[5 * nv] = on ? (float)s.w.z : 0.0f;
      }
  }
}

template <int NC>
hipError_t launch_class(const JacMassArgs& a, hipStream_t stream) {
  const size_t lds = (size_t)(JacLds<NC>::root + 13 * a.m.n_actors) * sizeof(R);
  hipLaunchKernelGGL(dense_jacmass_kernel<NC>, dim3(a.n_envs), dim3(64), lds, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dense_jacmass(const JacMassArgs& a, int nc, hipStream_t stream) {
  if (a.n_envs <= 0) return hipSuccess;
  return nc == 16 ? launch_class<16>(a, stream) : nc == 28 ? launch_class<28>(a, stream) : launch_class<32>(a, stream);
}

}  // namespace ags
