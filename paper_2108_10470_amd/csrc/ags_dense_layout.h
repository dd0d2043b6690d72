// LDS layout of the dense step kernel (one environment per 64-lane workgroup): plain C++ with no HIP
// dependency, shared by the host runtime and the host-side layout checker of the tests.
#pragma once

#include <algorithm>

#include "../../include/ags.h"

namespace ags {

constexpr int kDenseMaxV = 31;      // columns: one lane each below 32, and one more lane for the right-hand side
constexpr int kDenseMaxLinks = 32;  // links: one lane and one mask bit each
constexpr int kDenseRows = 64;      // rows solved one per lane; more go through global scratch
constexpr int kDenseChunk = 32;     // rows whose Jacobian columns are formed at a time
constexpr int kDenseLdsRows = 32;   // rows whose Delassus matrix is kept in LDS
constexpr int kDenseAStride = 33;   // its row stride (odd: its transposed tile is written without bank conflicts)
constexpr int kDenseXStride = 17;   // words per link of the subtree sums (10 inertia, 6 force; odd: no bank conflicts)
constexpr int kDensePose = 7;       // words per link pose: quaternion xyzw, origin

// offsets in words of the compute type, except the integer arrays (t_*, sact, slk, rkr, rm), which are in ints
struct DenseLds {
  int t_la, t_lcm, t_ccm;                   // model masks: ancestors of a link, columns moving a link, columns of a row of M
  int qj, qd, root, vs, lam, u, sact, slk, rkr, rm;  // live through a substep
  // dynamics region: column axes, link poses, link velocities (later the columns' momenta, then the rows' forces
  // of one chunk in pose and V), per-link sums (later the mass matrix); the Delassus matrix of at most
  // kDenseLdsRows rows overlays the region from its start, below the contact slots
  int S, pose, V, X, slots;
  int A;
  int G;      // packed columns of the inverse Cholesky factor's transpose (before them, a 1 among 63 zeros)
  int total;  // words of the compute type
};

inline DenseLds make_dense_layout(const ags_model_info& info, int n_tendon_joints, int elem_bytes) {
  DenseLds L{};
  const int ratio = elem_bytes / 4;
  const int nl = info.n_links, nv = info.n_v, nd = info.n_dof, na = info.n_actors, ns = info.n_slots;
  int off = 0;
  auto take = [&](int words) {
    const int o = off;
    off += (std::max(words, 1) + 1) & ~1;
    return o;
  };
  auto take_i = [&](int ints) { return take((std::max(ints, 1) + ratio - 1) / ratio) * ratio; };
  L.t_la = take_i(nl);
  L.t_lcm = take_i(nl);
  L.t_ccm = take_i(nv);
  L.qj = take(nd);
  L.qd = take(nv);
  L.root = take(13 * na);
  L.vs = take(nv);
  L.lam = take(kDenseRows);
  L.u = take(64);
  L.sact = take_i(ns);
  L.slk = take_i(ns);
  L.rkr = take_i(kDenseRows);
  L.rm = take_i(2 * kDenseRows);
  const int begin = off;
  L.A = begin;
  L.S = take(6 * nv);
  L.pose = take(kDensePose * nl);
  L.V = take(std::max(6 * std::max(nl, nv), 6 * kDenseChunk - kDensePose * nl));
  const int shared = off;
  L.X = take(std::max({kDenseXStride * nl, nv * (nv + 1) / 2 + 32, 6 * (nv + nl), 2 * n_tendon_joints}));
  const int x_end = off;
  off = std::max(shared, begin + kDenseLdsRows * kDenseAStride);
  L.slots = take(7 * ns);
  off = std::max(off, x_end);
  L.G = take(std::max(nv * (nv + 1) / 2, 64));
  L.total = off;
  return L;
}

}  // namespace ags
