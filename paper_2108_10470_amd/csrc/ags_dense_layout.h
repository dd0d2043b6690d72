// LDS layout of the dense step kernel (one environment per 64-lane workgroup): plain C++ with no HIP
// dependency, shared by the host runtime and the host-side layout checker of the tests.
#pragma once

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

// Size class of a model: NC - 1 columns and NC links at most, NC a multiple of four (the contraction step of a matrix
// tile).  The kernels are compiled per class, so that these offsets are constants and loops over columns and links have
// no bounds tests; columns and links past the model's are zeros.  28 is the humanoid's class (27 columns).
constexpr int dense_class(int n_v, int n_links) {
  return n_v <= 15 && n_links <= 16 ? 16 : n_v <= 27 && n_links <= 28 ? 28 : 32;
}

// offsets in 8-byte words, except the integer arrays (t_*, rkr, rm), which are in ints
template <int NC>
struct DenseLds {
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  // model masks: ancestors of a link, columns moving a link, columns of a row of M
  static constexpr int t_la = 0, t_lcm = NC, t_ccm = 2 * NC;
  // live through a substep
  static constexpr int qj = 3 * NC / 2, qd = qj + NC, vs = qd + NC, lam = vs + NC, u = lam + kDenseRows, rkr = 2 * (u + 64),
                       org = u + 64 + kDenseRows / 2;
  // dynamics region: column axes, link poses, link velocities (later the columns' momenta, then the rows' forces of
  // one chunk in pose and V), per-link sums (later the mass matrix, then the rows' column masks); the Delassus matrix
  // of at most kDenseLdsRows rows overlays the region from its start
  static constexpr int S = org + 4, pose = S + 6 * NC, V = pose + kDensePose * NC, X = V + 6 * NC,
                       x_words = max2(kDenseXStride * NC, NC * (NC + 1) / 2), rm = 2 * X, A = S;
  // pairs of columns of the factor's inverse transpose, column pair m as (2 m + 2) x 2 words (before them, a 1 among
  // 63 zeros)
  static constexpr int G = max2(X + x_words, A + kDenseLdsRows * kDenseAStride), g_words = NC / 2 * (NC / 2 + 1) * 2;
  static constexpr int fixed = G + g_words;  // then the model's root states and contact slots
  static_assert(G % 2 == 0 && u % 2 == 0, "16-byte aligned pairs");
  static_assert(kDensePose * NC + 6 * NC >= 6 * kDenseChunk && x_words >= kDenseRows, "overlaid arrays fit");
};

// the part that depends on the model, behind the class's fixed part
struct DenseDyn {
  int root;   // 13 words per actor
  int slots;  // normal (3 words), point (3) and distance of every slot, in three arrays
  int sact, slk;  // ints per slot: first row or -1; links
  int total;  // words
};

inline DenseDyn make_dense_layout(const ags_model_info& info, int fixed_words) {
  DenseDyn D{};
  int off = fixed_words;
  D.root = off;
  off += (13 * info.n_actors + 1) & ~1;
  D.slots = off;
  off += 7 * info.n_slots;
  D.sact = 2 * off;
  D.slk = D.sact + info.n_slots;
  off += info.n_slots;
  D.total = (off + 1) & ~1;
  return D;
}
inline int dense_fixed_words(int nc) {
  return nc == 16 ? DenseLds<16>::fixed : nc == 28 ? DenseLds<28>::fixed : DenseLds<32>::fixed;
}
inline int dense_x_words(int nc) {
  return nc == 16 ? DenseLds<16>::x_words : nc == 28 ? DenseLds<28>::x_words : DenseLds<32>::x_words;
}

}  // namespace ags
