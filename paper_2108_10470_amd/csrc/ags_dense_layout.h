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

constexpr int kDenseContacts = 21;  // contacts of an environment whose rows fit its lanes

// Offsets in 8-byte words, except the integer arrays (t_*, lrow, rm, clk), which are in ints.  The overlays keep a
// workgroup at 10-15 KB, so that the registers and not the LDS bound how many fit a CU.
template <int NC>
struct DenseLds {
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  // model masks: ancestors of a link, columns moving a link, columns of a row of M
  static constexpr int t_la = 0, t_lcm = NC, t_ccm = 2 * NC;
  // live through a substep: positions, rates, v* (before it, the right-hand side), limit rows, reference point
  static constexpr int qj = 3 * NC / 2, qd = qj + NC, vs = qd + NC, lrow = 2 * (vs + NC), org = vs + NC + 32;
  // Dynamics region.  S: column axes.  pose: link poses.  V: link velocities, the columns' momenta, the factor's
  // broadcast window, link velocities under v*.  X: per-link sums, the packed mass matrix and behind it a 1 among 63
  // zeros; later the rows' column masks (rm), the coefficients of the factor's columns (co), the contacts (normal,
  // point, distance, links) and the limit rows' biases.  The rows' forces of one chunk overlay pose and V.
  static constexpr int S = org + 4, pose = S + 6 * NC, V = pose + kDensePose * NC, X = V + 6 * NC, strip = X + NC * (NC + 1) / 2,
                       rm = 2 * X, co = X + 64, cn = X + 128, cx = cn + 66, cphi = cx + 66, clk = 2 * (cphi + 22),
                       lbias = cphi + 34,
                       x_words = max2(max2(kDenseXStride * NC, NC * (NC + 1) / 2 + 64), 128 + 66 + 66 + 34 + 64);
  // The Delassus matrix of at most kDenseLdsRows rows overlays the region from its start, after the sweeps the impulses
  // and the velocity change in the factor's columns.  G: pairs of columns of the factor's inverse transpose, column pair
  // m as (2 m + 2) x 2 words, behind the Delassus matrix (over the tail of X, written when the mass matrix has been read).
  static constexpr int A = S, lam = A, u = A + kDenseRows, G = A + kDenseLdsRows * kDenseAStride,
                       g_words = NC / 2 * (NC / 2 + 1) * 2;
  static constexpr int fixed = max2(X + x_words, G + g_words);  // then the model's root states
  static_assert(S % 2 == 0 && V % 2 == 0 && co % 2 == 0 && u % 2 == 0 && G % 2 == 0, "16-byte aligned pairs");
  static_assert(kDensePose * NC + 6 * NC >= 6 * kDenseChunk && 6 * NC >= 64, "overlaid arrays fit");
  static_assert(lbias + 64 <= G, "the factor's columns leave what is read after them alone");
};

struct DenseDyn {
  int root;   // 13 words per actor
  int total;  // words
};
inline DenseDyn make_dense_layout(const ags_model_info& info, int fixed_words) {
  return {fixed_words, (fixed_words + 13 * info.n_actors + 1) & ~1};
}
inline int dense_fixed_words(int nc) {
  return nc == 16 ? DenseLds<16>::fixed : nc == 28 ? DenseLds<28>::fixed : DenseLds<32>::fixed;
}
inline int dense_x_words(int nc) {
  return nc == 16 ? DenseLds<16>::x_words : nc == 28 ? DenseLds<28>::x_words : DenseLds<32>::x_words;
}

// LDS of the dense adjoint (RT tiles of 16 rows), offsets in 8-byte words except t_*, rm, lrow, clk, cel (ints).
template <int NC, int RT>
struct DenseAdjLds {
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  static constexpr int rows = 16 * RT, contacts = rows / 3;
  static constexpr int A_stride = rows + 1, Z_stride = 33;  // odd: columns are read without bank conflicts
  static constexpr int t_la = 0, t_lcm = NC, t_ccm = 2 * NC;
  // per column, 32 words each so that a lane group can step from one to the next: velocity change of the impulses,
  // z = M^-1 nubar, free acceleration, w = M^-1 h v*bar; v*, rates, positions, nubar, v*bar, rate adjoints
  static constexpr int dv = 3 * NC / 2, z = dv + 32, qdd = z + 32, w = qdd + 32, vs = w + 32, nu = vs + 32, qj = nu + 32,
                       nub = qj + 32, vsb = nub + 32, nui = vsb + 32, u = nui + 32, nh = u + 64, uh = nh + 32, org = uh + 32;
  // kept from the recomputation: column axes, link poses, velocities, accelerations, composite inertias, momenta, factor
  static constexpr int Ic_stride = 11;
  static constexpr int S = org + 4, pose = S + 6 * NC + (6 * (32 - NC)), V = pose + kDensePose * NC, Acc = V + 6 * NC,
                       Ic = Acc + 6 * NC, Fm = Ic + Ic_stride * NC, G = Fm + 6 * 32, g_words = NC / 2 * (NC / 2 + 1) * 2,
                       co = G + g_words;
  // rows: forces (before them the factor's window, after them the contacts' wrenches), masks, impulses and their adjoints
  static constexpr int rowf = co + 64, rm = 2 * (rowf + 6 * rows), lamy = rowf + 7 * rows, lbias = lamy + 2 * rows,
                       lrow = 2 * (lbias + 64), cn = lbias + 64 + 32, cx = cn + 3 * contacts, cphi = cx + 3 * contacts,
                       clk = 2 * (cphi + contacts), cel = clk + 2 * ((contacts + 1) / 2),
                       work = (cel / 2 + contacts + 3) & ~1;
  // work: per-link sums and records (17 words each, twice), the packed mass matrix, the Delassus matrix, rows x columns
  // products, the column adjoint matrix
  static constexpr int work_words = max2(max2(rows * A_stride, max2(rows, 32) * Z_stride), 34 * 32);
  static constexpr int fixed = (work + work_words + 1) & ~1;
  static_assert(S % 2 == 0 && G % 2 == 0 && co % 2 == 0 && rowf % 2 == 0 && u % 2 == 0 && work % 2 == 0, "16-byte aligned pairs");
  static_assert(NC * (NC + 1) / 2 + 64 <= work_words && 6 * (2 * contacts + 4) <= 6 * rows, "overlaid arrays fit");
};

struct DenseAdjDyn {
  int tape;                    // per sweep and row: change of the impulse, then (reverse) the row adjoint after the sweep
  int iters4;                  // sweeps, rounded up to the contraction step of a tile
  int mask;                    // per sweep: bits of the rows updated freely, of those at the upper bound
  int st, rbar, nrb, dbar;     // state at every substep's start; adjoints of roots, of their pose, of DOFs
  int state_words, rows_cap, total;
};
inline DenseAdjDyn make_dense_adj_layout(const ags_model_info& info, int substeps, int iters, int row_cap, int fixed_words,
                                         int rows) {
  DenseAdjDyn d{};
  d.iters4 = (iters + 3) & ~3;
  int off = fixed_words;
  auto take = [&](int n) {
    const int o = off;
    off += (n + 1) & ~1;
    return o;
  };
  d.tape = take(2 * d.iters4 * rows > 192 ? 2 * d.iters4 * rows : 192);
  d.mask = take(2 * d.iters4);
  d.state_words = 13 * info.n_actors + 2 * info.n_dof;
  d.st = take(substeps * d.state_words);
  d.rbar = take(13 * info.n_actors);
  d.nrb = take(13 * info.n_actors);
  d.dbar = take(2 * info.n_dof);
  const int rc = info.max_rows > 1 ? info.max_rows : 1;
  d.rows_cap = rc < row_cap ? rc : row_cap;
  d.total = off;
  return d;
}
inline int dense_adj_fixed_words(int nc, int big) {
  return nc == 16   ? (big ? DenseAdjLds<16, 4>::fixed : DenseAdjLds<16, 2>::fixed)
         : nc == 28 ? (big ? DenseAdjLds<28, 4>::fixed : DenseAdjLds<28, 2>::fixed)
                    : (big ? DenseAdjLds<32, 4>::fixed : DenseAdjLds<32, 2>::fixed);
}

}  // namespace ags
